// Triples -> subject-indexed CSR on gfx950.
//
// The CSR's rows must keep the triples' input order (a stable sort by subject),
// so that walk parity is exact and independent of scheduling. Atomics cannot
// give that order; an LSD radix sort on the subject id can, because every pass
// is a stable counting sort on one digit. A pass is three launches:
//   1. radix_count:   per tile of up to 8,192 triples, a histogram of the pass's digit
//                     (LDS atomics), written digit-major to a count table;
//   2. row_scan:      exclusive scan of each digit's row of that table (one
//                     workgroup per digit) and the digit's total;
//   3. radix_scatter: per tile, the stable rank of every triple among the
//                     tile's triples with the same digit (wave ballots give the
//                     lanes sharing a digit, per-wave LDS counters carry the
//                     count across rounds), a local reorder through LDS, then
//                     writes of runs of equal digits to their global slots.
// The first pass also checks every id range. row_ptr comes from one pass over
// the sorted subjects, so no kernel needs global atomics (power-law hubs would
// serialise them). Up to one tile of triples over few entities is sorted by a
// single workgroup in one launch (csr_small_kernel).
//
// What bounds a pass is HBM traffic (12 B read and written per triple), so the
// sort takes as few passes as possible: digits of up to 10 bits, against a
// tile of 8,192 triples that keeps the runs of a 1,024-bin pass at 8 triples.
// 20M triples over 1M entities: two passes of 10 bits, 120 + 106 us of scatter
// (4.0 TB/s), against 100 + 2 x 96 us for 7, 7 and 6 bits in 4,096-triple
// tiles; with count, scan and row_ptr 322 us against 418. 500M over 50M: 9, 7
// and 10 bits, 2.75 + 2.49 + 2.61 ms, against 10.1 ms in four passes.
// The last pass sorts by the top digit, whose value follows from the position,
// so it writes only the low 16 bits of the subjects (or none if there are no
// lower bits).
//
// Workspace: two key buffers (4 B/triple each), one payload buffer (8 B/triple;
// edges_out is the other), the count table and the digit totals. The wide
// tables of the first and the last pass lie in parts of the key buffers those
// passes leave free.

#include <algorithm>

#include "common.hpp"
#include "launch.hpp"
#include "xcd.hpp"

namespace rdf2v {
namespace {

typedef int32_t v2i32 __attribute__((ext_vector_type(2)));

// A tile is kSortThreads triples per round and kRounds rounds (2, 4 or 8; the
// plan picks one): wave w of its workgroup owns kRounds * 64 consecutive
// triples, taken 64 a round.
constexpr int kSortThreads = 1024;
constexpr int kMostRounds = 8;
constexpr int kMostTile = kSortThreads * kMostRounds;
constexpr int kMaxDigitBits = 10;
constexpr int kMaxBins = 1 << kMaxDigitBits;
constexpr int kTileWaves = kSortThreads / kWave;

static_assert(kMaxBins <= kSortThreads, "one thread per digit in the tile prefix step");
static_assert(kMostTile <= 65535, "positions inside a tile are kept in 16 bits");

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
// Entries per digit in the count table: the tiles, padded so that a row starts 16-byte aligned.
__host__ __device__ inline int64_t row_stride(int64_t tiles) { return (tiles + 3) / 4 * 4; }

// ---------------------------------------------------------------------------
// Radix pass, step 1: per-tile digit histogram (+ subject id validation on
// pass 0; the first scatter, which reads predicates and objects anyway,
// validates those). Pass 0 also marks every row_ptr entry as not yet known.
// ---------------------------------------------------------------------------
// Each thread reads kCountItems keys as 16-byte vectors (all loads issued
// before any histogram update) and counts them in LDS.
constexpr int kCountThreads = 256;

template <bool kFirst, int kRounds>
__global__ __launch_bounds__(kCountThreads) void radix_count_kernel(
    const uint32_t *__restrict__ keys, int64_t n, int shift, int bits, int32_t num_entities,
    int32_t *__restrict__ counts, int64_t tiles, int32_t *__restrict__ row_ptr, int32_t *status) {
  __shared__ int hist[kMaxBins];
  constexpr int kTile = kSortThreads * kRounds;
  constexpr int kCountItems = kTile / kCountThreads;  // keys per thread
  constexpr int kVec = 4;
  constexpr int kLoads = kCountItems / kVec;
  const int bins = 1 << bits;
  const uint32_t mask = uint32_t(bins - 1);
  const int64_t tile = xcd_tile(blockIdx.x, tiles);
  const int64_t base = tile * kTile;
  const bool full = base + kTile <= n && (reinterpret_cast<uintptr_t>(keys) & 15) == 0;
  uint32_t k[kCountItems];
  if (full) {
    // 16-byte loads: vector v of the tile holds keys 4v .. 4v+3.
    const uint4 *k4 = reinterpret_cast<const uint4 *>(keys + base);
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const uint4 v = k4[i * kCountThreads + threadIdx.x];
      k[kVec * i + 0] = v.x; k[kVec * i + 1] = v.y; k[kVec * i + 2] = v.z; k[kVec * i + 3] = v.w;
    }
  }
  for (int i = threadIdx.x; i < bins; i += kCountThreads) hist[i] = 0;
  if (kFirst && row_ptr != nullptr) {
    const int64_t nv = int64_t(num_entities) + 1;
    for (int64_t v = int64_t(blockIdx.x) * kCountThreads + threadIdx.x; v < nv; v += int64_t(gridDim.x) * kCountThreads)
      row_ptr[v] = -1;
  }
  __syncthreads();
  int bad = 0;
  if (full) {
    if (kFirst) {
#pragma unroll
      for (int i = 0; i < kCountItems; ++i) bad |= k[i] >= uint32_t(num_entities);
    }
    // After the first pass the keys of a tile are grouped by their lower digits, and in
    // power-law graphs many tiles hold one hub's triples only: a wave's 64 increments of one
    // bin would serialise on one LDS address. The lanes that share lane 0's digit add their
    // number with one atomic instead.
    const int lane = lane_id();
#pragma unroll
    for (int i = 0; i < kCountItems; ++i) {
      const uint32_t d = (k[i] >> shift) & mask;
      const uint32_t d0 = __builtin_amdgcn_readfirstlane(d);
      const uint64_t same = __ballot(d == d0);
      if (d != d0)
        atomicAdd(&hist[d], 1);
      else if (lane == 0)
        atomicAdd(&hist[d0], __popcll(same));
    }
  } else {
    // ragged last tile or unaligned input: scalar loads of the same items
    for (int i = 0; i < kCountItems; ++i) {
      const int64_t idx = base + int64_t(i / kVec) * (kCountThreads * kVec) + threadIdx.x * kVec + (i % kVec);
      if (idx < n) {
        const uint32_t key = keys[idx];
        atomicAdd(&hist[(key >> shift) & mask], 1);
        if (kFirst) bad |= key >= uint32_t(num_entities);
      }
    }
  }
  if (kFirst) {
    if (__syncthreads_or(bad) && threadIdx.x == 0 && status != nullptr)
      atomicOr(status, RDF2V_STATUS_ID_OUT_OF_RANGE);
  } else {
    __syncthreads();
  }
  const int64_t stride = row_stride(tiles);
  for (int d = threadIdx.x; d < bins; d += kCountThreads) counts[int64_t(d) * stride + tile] = hist[d];
}

// ---------------------------------------------------------------------------
// Radix pass, step 2: workgroup d scans digit d's counts over the tiles, in
// place, and writes the digit's total. (The scatter's workgroups add the
// totals of the lower digits themselves.)
// ---------------------------------------------------------------------------
constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanTile = kScanThreads * kScanItems;

__global__ __launch_bounds__(kScanThreads) void row_scan_kernel(int32_t *__restrict__ counts, int64_t tiles,
                                                                int32_t *__restrict__ totals) {
  __shared__ int scratch[kScanThreads / kWave];
  int32_t *row = counts + int64_t(blockIdx.x) * row_stride(tiles);
  int carry = 0;
  for (int64_t base = 0; base < tiles; base += kScanTile) {
    const int64_t i0 = base + int64_t(threadIdx.x) * kScanItems;
    int v[kScanItems];
#pragma unroll
    for (int k = 0; k < kScanItems; k += 4) {
      int4 x = make_int4(0, 0, 0, 0);
      if (i0 + k < tiles) x = *reinterpret_cast<const int4 *>(row + i0 + k);  // rows are padded to 4
      v[k] = x.x; v[k + 1] = x.y; v[k + 2] = x.z; v[k + 3] = x.w;
    }
    int sum = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) sum += i0 + k < tiles ? v[k] : 0;
    int tot;
    int ex = carry + block_exclusive_scan<kScanThreads>(sum, scratch, tot);
#pragma unroll
    for (int k = 0; k < kScanItems; k += 4) {
      int4 x;
      x.x = ex; ex += v[k];
      x.y = ex; ex += v[k + 1];
      x.z = ex; ex += v[k + 2];
      x.w = ex; ex += v[k + 3];
      if (i0 + k < tiles) *reinterpret_cast<int4 *>(row + i0 + k) = x;
    }
    carry += tot;
  }
  if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

// ---------------------------------------------------------------------------
// Radix pass, step 3: stable scatter of one tile.
// ---------------------------------------------------------------------------

// Exclusive scan over the block of two int32 values per thread at once.
template <int NT>
__device__ __forceinline__ int2 block_exclusive_scan2(int2 x, int2 *scratch) {
  constexpr int kWaves = NT / kWave;
  const int lane = lane_id();
  const int wave = threadIdx.x / kWave;
  int2 v = x;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int a = __shfl_up(v.x, off, kWave), b = __shfl_up(v.y, off, kWave);
    if (lane >= off) {
      v.x += a;
      v.y += b;
    }
  }
  if (lane == kWave - 1) scratch[wave] = v;
  __syncthreads();
  // sums of the waves before: one wave total per lane, added over the lanes below `wave`
  int2 before = lane < wave ? scratch[lane] : make_int2(0, 0);
#pragma unroll
  for (int off = 1; off < kWaves; off <<= 1) {
    before.x += __shfl_xor(before.x, off, kWave);
    before.y += __shfl_xor(before.y, off, kWave);
  }
  before.x = __builtin_amdgcn_readfirstlane(before.x);
  before.y = __builtin_amdgcn_readfirstlane(before.y);
  return make_int2(before.x + v.x - x.x, before.y + v.y - x.y);
}

// Position of each of the thread's items (item r of wave w: (w * kRounds + r)
// * 64 + lane) in the tile's stable order by the digit (key >> shift) & (bins
// - 1), and for thread d < bins the tile-local start of digit d (x) and the sum
// of `total` over the lower digits (y). kBits >= the digit's bits.
// wave_count: kTileWaves * bins counters, zeroed here; they and digit_start
// (one per digit) are free again after the barrier that the caller puts behind
// the call.
template <int kBits, int kRounds>
__device__ __forceinline__ int2 tile_positions(const uint32_t (&key)[kRounds], int tile_n, int shift, int bins,
                                               int total, uint16_t *wave_count, int *digit_start, int2 *scratch,
                                               uint32_t (&pos)[kRounds]) {
  const uint32_t mask = uint32_t(bins - 1);
  const int lane = lane_id();
  const int wave = threadIdx.x / kWave;
  for (int i = threadIdx.x; i < kTileWaves * bins / 2; i += kSortThreads) reinterpret_cast<uint32_t *>(wave_count)[i] = 0;
  __syncthreads();
  uint16_t *mine = wave_count + wave * bins;
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const bool valid = (wave * kRounds + r) * kWave + lane < tile_n;
    const uint32_t d = (key[r] >> shift) & mask;
    const uint32_t before = valid ? mine[d] : 0;
    // Lanes of this round holding the same digit: per bit, the lanes whose bit
    // is the lane's own (in halves: four instructions a bit).
    const uint64_t all = __ballot(valid);
    uint32_t lo = uint32_t(all), hi = uint32_t(all >> 32);
#pragma unroll
    for (int b = 0; b < kBits; ++b) {
      const uint32_t own = uint32_t(int32_t(d << (31 - b)) >> 31);  // the lane's bit in every position
      const uint64_t m = __ballot(own != 0);
      lo &= ~(uint32_t(m) ^ own);
      hi &= ~(uint32_t(m >> 32) ^ own);
    }
    const uint32_t below = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
    pos[r] = before + below;
    // The lowest lane of each digit group advances the wave's counter; its
    // store depends on the load above, so every lane's load precedes it.
    if (valid && below == 0) mine[d] = uint16_t(before + __popc(lo) + __popc(hi));
    __builtin_amdgcn_sched_barrier(0);  // one round's masks in registers at a time
  }
  __syncthreads();
  // Tile-local start of every (wave, digit) run.
  const int d = threadIdx.x;
  int sum = 0;
  if (d < bins) {
#pragma unroll
    for (int w = 0; w < kTileWaves; ++w) {  // counts -> starts within the digit
      const int c = wave_count[w * bins + d];
      wave_count[w * bins + d] = uint16_t(sum);
      sum += c;
    }
  }
  const int2 start = block_exclusive_scan2<kSortThreads>(make_int2(sum, total), scratch);
  if (d < bins) digit_start[d] = start.x;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    // min: always inside the tile; keeps a logic slip from leaving the tile
    const uint32_t dr = (key[r] >> shift) & mask;
    pos[r] = min(uint32_t(digit_start[dr]) + mine[dr] + pos[r], uint32_t(kSortThreads * kRounds - 1));
  }
  return start;
}

// Bytes of LDS that the counters, the keys and the payloads of a tile use in turn.
template <int kRounds>
constexpr int kStageBytes = kSortThreads * kRounds * 8 > kTileWaves * kMaxBins * 2 ? kSortThreads * kRounds * 8
                                                                                   : kTileWaves * kMaxBins * 2;

// kKeyOut: how the pass writes its keys: 4 B each, their low 16 bits (the last
// pass: keys_out is then a uint16_t array), or not at all (0).
template <bool kFirst, int kKeyOut, int kBits, int kRounds>
__global__ __launch_bounds__(kSortThreads) __attribute__((amdgpu_waves_per_eu(8))) void radix_scatter_kernel(
    const uint32_t *__restrict__ keys_in, const int2 *__restrict__ pay_in,
    const int32_t *__restrict__ pred_in, const int32_t *__restrict__ obj_in,
    void *__restrict__ keys_out, int2 *__restrict__ pay_out, int64_t n, int shift, int bits,
    const int32_t *__restrict__ offsets, const int32_t *__restrict__ totals, int32_t *__restrict__ bases_out,
    int64_t tiles, int32_t num_entities, int32_t num_predicates, int32_t *status) {
  constexpr int kTile = kSortThreads * kRounds;
  __shared__ __align__(16) char stage[kStageBytes<kRounds>];
  __shared__ int digit_start[kMaxBins];
  __shared__ int2 scan_scratch[kSortThreads / kWave];
  const int bins = 1 << bits;
  const uint32_t mask = uint32_t(bins - 1);
  const int lane = lane_id();
  const int wave = threadIdx.x / kWave;
  const int64_t tile = xcd_tile(blockIdx.x, tiles);
  const int64_t base = tile * kTile;
  const int tile_n = int(min(int64_t(kTile), n - base));

  // Inputs are read once, past the caches (non-temporal), which leaves L2 to
  // the lines that neighbouring tiles fill together: 127 -> 120 and 119 -> 106
  // us for the two passes over 20M triples.
  // The wave's keys are loaded together, with thread d's start of digit d among
  // the tiles and the digit's total; its payloads after the ranking (64
  // registers hold no more), in flight while the keys are written.
  uint32_t key[kRounds];
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const int local = (wave * kRounds + r) * kWave + lane;
    key[r] = local < tile_n ? __builtin_nontemporal_load(keys_in + base + local) : 0;
  }
  const int32_t digit_offset = threadIdx.x < bins ? offsets[int64_t(threadIdx.x) * row_stride(tiles) + tile] : 0;
  const int32_t digit_total = threadIdx.x < bins ? totals[threadIdx.x] : 0;

  uint32_t pos[kRounds];
  const int2 start = tile_positions<kBits, kRounds>(key, tile_n, shift, bins, digit_total,
                                           reinterpret_cast<uint16_t *>(stage), digit_start, scan_scratch, pos);
  int2 pay[kRounds];
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const int local = (wave * kRounds + r) * kWave + lane;
    pay[r] = make_int2(0, 0);
    if (local < tile_n) {
      if (kFirst) {
        pay[r] = make_int2(__builtin_nontemporal_load(pred_in + base + local), __builtin_nontemporal_load(obj_in + base + local));
      } else {
        const v2i32 v = __builtin_nontemporal_load(reinterpret_cast<const v2i32 *>(pay_in + base) + local);
        pay[r] = make_int2(v.x, v.y);
      }
    }
  }
  __syncthreads();
  int *global_minus_local = digit_start;
  if (threadIdx.x < bins) {
    global_minus_local[threadIdx.x] = start.y + digit_offset - start.x;
    if (bases_out != nullptr && blockIdx.x == 0) bases_out[threadIdx.x] = start.y;
  }
  // The keys through LDS first, then the payloads through the same bytes: 68 KB
  // of LDS in all, so two workgroups share a CU and one ranks while the other
  // loads or writes.
  uint32_t *s_keys = reinterpret_cast<uint32_t *>(stage);
#pragma unroll
  for (int r = 0; r < kRounds; ++r)
    if ((wave * kRounds + r) * kWave + lane < tile_n) s_keys[pos[r]] = key[r];
  __syncthreads();
  int32_t to[kRounds];  // global slot of tile position threadIdx.x + i * kSortThreads
#pragma unroll
  for (int i = 0; i < kRounds; ++i) {
    const int j = threadIdx.x + i * kSortThreads;
    to[i] = -1;
    if (j < tile_n) {
      const uint32_t k = s_keys[j];
      const uint32_t g = uint32_t(global_minus_local[(k >> shift) & mask] + j);
      if (g < uint32_t(n)) {  // always true for consistent counts; never write outside the arrays
        to[i] = int32_t(g);
        if (kKeyOut == 4) static_cast<uint32_t *>(keys_out)[g] = k;
        if (kKeyOut == 2) static_cast<uint16_t *>(keys_out)[g] = uint16_t(k);
      }
    }
    if (i % 2 == 1) __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();
  if (kFirst) {  // predicate and object ids (subjects were checked by the count pass)
    int bad = 0;
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
      bad |= (uint32_t(pay[r].x) >= uint32_t(num_predicates)) | (uint32_t(pay[r].y) >= uint32_t(num_entities));
    if (__ballot(bad) != 0 && lane == 0 && status != nullptr) atomicOr(status, RDF2V_STATUS_ID_OUT_OF_RANGE);
  }
  int2 *s_pay = reinterpret_cast<int2 *>(stage);
#pragma unroll
  for (int r = 0; r < kRounds; ++r)
    if ((wave * kRounds + r) * kWave + lane < tile_n) s_pay[pos[r]] = pay[r];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kRounds; ++i)
    if (to[i] >= 0) pay_out[uint32_t(to[i])] = s_pay[threadIdx.x + i * kSortThreads];
}

// ---------------------------------------------------------------------------
// One workgroup, one launch: at most kMostTile triples. The passes exchange keys
// and payloads through LDS. With row_ptr (at most kSmallEntities entities) it
// becomes the scan of a histogram of the subjects; else the sorted subjects go
// to keys_out for the row_ptr kernels. What bounds it is the chain of LDS
// round trips and barriers; the passes as kernels of their own would be bound
// by the gaps between thirteen launches (5,000 triples over 1,000
// entities: 14.6 us of kernel time in one launch, against 48 us in thirteen).
// ---------------------------------------------------------------------------
constexpr int kSmallEntities = kStageBytes<kMostRounds> / 4;

__global__ __launch_bounds__(kSortThreads) void csr_small_kernel(
    const uint32_t *__restrict__ subj, const int32_t *__restrict__ pred, const int32_t *__restrict__ obj, int n,
    int32_t num_entities, int32_t num_predicates, int total_bits, int32_t *__restrict__ row_ptr,
    int2 *__restrict__ edges, uint32_t *__restrict__ keys_out, int32_t *status) {
  constexpr int kRounds = kMostRounds;
  __shared__ __align__(16) char stage[kStageBytes<kRounds>];
  __shared__ int digit_start[kMaxBins];
  __shared__ int2 scan_scratch[kSortThreads / kWave];
  const bool with_row_ptr = row_ptr != nullptr;
  const int lane = lane_id();
  const int wave = threadIdx.x / kWave;
  uint32_t key[kRounds];
  int2 pay[kRounds];
  bool valid[kRounds];
  int bad = 0;
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const int i = (wave * kRounds + r) * kWave + lane;
    valid[r] = i < n;
    key[r] = 0;
    pay[r] = make_int2(0, 0);
    if (valid[r]) {
      key[r] = subj[i];
      pay[r] = make_int2(pred[i], obj[i]);
      bad |= (key[r] >= uint32_t(num_entities)) | (uint32_t(pay[r].x) >= uint32_t(num_predicates)) |
             (uint32_t(pay[r].y) >= uint32_t(num_entities));
    }
  }
  if (__ballot(bad) != 0 && lane == 0 && status != nullptr) atomicOr(status, RDF2V_STATUS_ID_OUT_OF_RANGE);

  if (with_row_ptr) {
    const int per = (num_entities + kSortThreads - 1) / kSortThreads;  // consecutive entities per thread
    int *hist = reinterpret_cast<int *>(stage);
    for (int v = threadIdx.x; v < per * kSortThreads; v += kSortThreads) hist[v] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
      if (valid[r] && key[r] < uint32_t(num_entities)) atomicAdd(&hist[key[r]], 1);
    __syncthreads();
    int sum = 0;
    for (int i = 0; i < per; ++i) sum += hist[threadIdx.x * per + i];
    int before = block_exclusive_scan2<kSortThreads>(make_int2(sum, 0), scan_scratch).x;
    for (int i = 0; i < per; ++i) {
      const int v = threadIdx.x * per + i;
      if (v < num_entities) row_ptr[v] = before;
      before += hist[v];
    }
    if (threadIdx.x == 0) row_ptr[num_entities] = n;
    __syncthreads();
  }

  const int passes = (total_bits + kMaxDigitBits - 1) / kMaxDigitBits;  // at most four
  for (int pass = 0, shift = 0; pass < passes; ++pass) {
    const int bits = (total_bits - shift + passes - pass - 1) / (passes - pass);
    uint32_t pos[kRounds];
    tile_positions<kMaxDigitBits, kRounds>(key, n, shift, 1 << bits, 0, reinterpret_cast<uint16_t *>(stage), digit_start, scan_scratch,
                      pos);
    __syncthreads();
    uint32_t *s_keys = reinterpret_cast<uint32_t *>(stage);
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
      if (valid[r]) s_keys[pos[r]] = key[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRounds; ++r) key[r] = valid[r] ? s_keys[(wave * kRounds + r) * kWave + lane] : 0;
    __syncthreads();
    int2 *s_pay = reinterpret_cast<int2 *>(stage);
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
      if (valid[r]) s_pay[pos[r]] = pay[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
      if (valid[r]) pay[r] = s_pay[(wave * kRounds + r) * kWave + lane];
    __syncthreads();
    shift += bits;
  }
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const int i = (wave * kRounds + r) * kWave + lane;
    if (valid[r]) edges[i] = pay[r];
    if (valid[r] && !with_row_ptr) keys_out[i] = key[r];
  }
}

// ---------------------------------------------------------------------------
// row_ptr[v] = number of sorted subjects < v, for v in [0, V], from the sorted
// subjects in one pass: where the subject changes from a (at position i-1) to
// b (at i), every v in (a, b] has row_ptr[v] = i; the subjects v above the
// last one get n. A thread writes at most gap_run of those entries; longer
// runs of entities without out-edges keep the -1 that the first count pass put
// there, and row_ptr_fixup_kernel finds each of them by binary search.
// ---------------------------------------------------------------------------
// Writing a gap is cheaper than a search per entry while the gaps are short
// or there are threads enough: 1M triples over 10M entities 144 us with runs
// of 64, 195 us with 1; 3M over 10M is slower with 1 as well. With four
// entities per triple and few triples, the threads that write the gaps, 16 of
// them each, are few and the searching ones many: 20,000 triples over 1M
// entities 175 us with runs of 64, 106 us with 1; 8,193 over 1M 161 / 63;
// 200,000 over 10M 214 / 148; 400,000 over 10M 181 / 165.
constexpr int kGapRun = 64;
constexpr int64_t kSparse = 4;                   // entities per triple ...
constexpr int64_t kSparseMax = int64_t(1) << 19;  // ... and fewer triples than this: runs of 1

// The sorted subjects as the last pass left them: the low bits of each, and
// where each top digit begins. kKey: bytes of a stored key (4: the whole
// subject, and the digits are not used; 2; 0: there are no low bits).
struct SortedKeys {
  const void *keys;
  const int32_t *bases;  // [bins]
  int bins;
  int low_bits;
};

template <int kKey>
__device__ __forceinline__ uint32_t stored_key(const SortedKeys &k, int64_t i) {
  if (kKey == 4) return static_cast<const uint32_t *>(k.keys)[i];
  if (kKey == 2) return static_cast<const uint16_t *>(k.keys)[i] & ((1u << k.low_bits) - 1);
  return 0;
}

// Each thread takes consecutive positions (two 16-byte loads of keys). The top
// digit of a wave's first position comes from two ballots over the bases; where
// none begins among the wave's positions, as nearly everywhere, that is the
// digit of them all. (A search per thread through the bases in LDS took 32 us
// at 20M triples, twice the 4-byte keys' time.)
constexpr int kBoundThreads = 256;
template <int kKey>
constexpr int kBoundItems = kKey == 4 ? 8 : 16;

template <int kKey>
__global__ __launch_bounds__(kBoundThreads) void row_ptr_bounds_kernel(const SortedKeys sorted,
                                                                       int64_t n_triples, int32_t num_entities,
                                                                       uint32_t gap_run,
                                                                       int32_t *__restrict__ row_ptr) {
  // Positions and ids are below 2^31: unsigned 32-bit arithmetic throughout.
  constexpr uint32_t kItems = kBoundItems<kKey>;
  const uint32_t n = uint32_t(n_triples), V = uint32_t(num_entities);
  const uint32_t lane = uint32_t(lane_id());
  const uint32_t w0 = (blockIdx.x * uint32_t(kBoundThreads) + threadIdx.x - lane) * kItems;  // the wave's first
  if (w0 > n) return;  // uniform per wave
  const uint32_t i0 = w0 + lane * kItems;
  uint32_t k[kItems];
  if (i0 + kItems <= n && (reinterpret_cast<uintptr_t>(sorted.keys) & 15) == 0 && kKey != 0) {
    const uint4 *k4 = reinterpret_cast<const uint4 *>(static_cast<const char *>(sorted.keys) + size_t(i0) * kKey);
    const uint4 v[2] = {k4[0], k4[1]};
#pragma unroll
    for (uint32_t j = 0; j < 2; ++j) {
      const uint32_t w[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
#pragma unroll
      for (uint32_t c = 0; c < 4; ++c) {
        if (kKey == 4) {
          k[4 * j + c] = w[c];
        } else {
          const uint32_t low = (1u << sorted.low_bits) - 1;
          k[(8 * j + 2 * c) % kItems] = w[c] & low;
          k[(8 * j + 2 * c + 1) % kItems] = (w[c] >> 16) & low;
        }
      }
    }
  } else {
#pragma unroll
    for (uint32_t j = 0; j < kItems; ++j) k[j] = i0 + j < n ? stored_key<kKey>(sorted, i0 + j) : 0u;
  }
  const uint32_t prev = i0 > 0 && i0 <= n ? stored_key<kKey>(sorted, i0 - 1) : 0u;
  uint32_t d = 0;  // top digit of position i0 - 1, then of each position in turn
  uint32_t next = 0xffffffffu;  // where digit d + 1 begins
  if (kKey != 4) {
    // largest digit whose base is at or below `at`: 64 samples, then the bases between two of them
    const uint32_t bins = uint32_t(sorted.bins);
    const uint32_t *bases = reinterpret_cast<const uint32_t *>(sorted.bases);
    const uint32_t at = min(w0 > 0 ? w0 - 1 : 0u, n - 1);
    const uint32_t step = max(1u, bins / kWave);  // bins is a power of two, at most 1024
    const uint32_t s = (__popcll(__ballot(lane * step < bins && bases[min(lane * step, bins - 1)] <= at)) - 1) * step;
    d = s + __popcll(__ballot(lane < step && bases[min(s + lane, bins - 1)] <= at)) - 1;
    next = d + 1 < bins ? bases[d + 1] : 0xffffffffu;
    const uint32_t before = min(i0 > 0 ? i0 - 1 : 0u, n - 1);
    while (next <= before) {
      ++d;
      next = d + 1 < bins ? bases[d + 1] : 0xffffffffu;
    }
  }
  if (i0 > n) return;
  // entities in (a, b] start at position i; a = -1 before the first subject, b = V after the last
  auto whole = [&](uint32_t low) -> uint32_t { return kKey == 4 ? low : (d << sorted.low_bits) | low; };
  uint32_t first = i0 == 0 ? 0u : whole(prev) + 1;  // a + 1
#pragma unroll
  for (uint32_t j = 0; j < kItems; ++j) {
    const uint32_t i = i0 + j;
    if (i > n) break;
    while (next <= i && i < n) {
      ++d;
      next = d + 1 < uint32_t(sorted.bins) ? uint32_t(sorted.bases[d + 1]) : 0xffffffffu;
    }
    const uint32_t b = i == n ? V : whole(k[j]);
    if (b >= first) {
      const uint32_t hi = min(b, V);  // ids >= V cannot occur after validation
      const uint32_t lo = max(first, hi >= gap_run ? hi - (gap_run - 1) : 0u);
      for (uint32_t v = lo; v <= hi; ++v) row_ptr[v] = int32_t(i);
    }
    first = b + 1;
  }
}

template <int kKey>
__global__ __launch_bounds__(256) void row_ptr_fixup_kernel(const SortedKeys sorted, int64_t n, int32_t num_entities,
                                                            int32_t *__restrict__ row_ptr) {
  const int64_t v = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (v > num_entities || row_ptr[v] >= 0) return;
  int64_t lo = 0, hi = n;
  uint32_t want = uint32_t(v);
  if (kKey != 4) {  // inside the range of v's top digit
    const int64_t d = v >> sorted.low_bits;
    lo = d < sorted.bins ? sorted.bases[d] : n;
    hi = d + 1 < sorted.bins ? int64_t(sorted.bases[d + 1]) : n;
    want &= (1u << sorted.low_bits) - 1;
  }
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (stored_key<kKey>(sorted, mid) < want) lo = mid + 1;
    else hi = mid;
  }
  row_ptr[v] = int32_t(lo);
}

__global__ __launch_bounds__(256) void fill_kernel(int32_t *p, int64_t n, int32_t value) {
  const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (i < n) p[i] = value;
}

// ---------------------------------------------------------------------------
// Entities with out-degree >= 1, ascending: a count per block of kStartTile
// entities (one launch, left out when there is one block only), then each block
// adds the counts before its own and writes its entities.
// ---------------------------------------------------------------------------
constexpr int kStartThreads = 1024;
constexpr int kStartItems = 16;
constexpr int kStartTile = kStartThreads * kStartItems;
constexpr int kStartWaves = kStartThreads / kWave;

// Bit i: entity v0 + i * 64 + lane of the calling wave has out-edges (v0 = the
// wave's first of kStartItems * 64 entities).
__device__ __forceinline__ uint32_t nonsink_flags(const int32_t *__restrict__ row_ptr, int32_t num_entities, int64_t v0) {
  int32_t lo[kStartItems], hi[kStartItems];
#pragma unroll
  for (int i = 0; i < kStartItems; ++i) {
    const int64_t v = v0 + i * kWave + lane_id();
    lo[i] = hi[i] = 0;
    if (v < num_entities) {
      lo[i] = row_ptr[v];
      hi[i] = row_ptr[v + 1];
    }
  }
  uint32_t f = 0;
#pragma unroll
  for (int i = 0; i < kStartItems; ++i) f |= hi[i] > lo[i] ? 1u << i : 0u;
  return f;
}

__global__ __launch_bounds__(kStartThreads) void nonsink_count_kernel(const int32_t *__restrict__ row_ptr,
                                                                      int32_t num_entities,
                                                                      int32_t *__restrict__ partials) {
  __shared__ int scratch[kStartWaves];
  const int64_t v0 = int64_t(blockIdx.x) * kStartTile + int64_t(threadIdx.x / kWave) * kWave * kStartItems;
  const int total = block_sum<kStartThreads, int>(int(__popc(nonsink_flags(row_ptr, num_entities, v0))), scratch);
  if (threadIdx.x == 0) partials[blockIdx.x] = total;
}

__global__ __launch_bounds__(kStartThreads) void nonsink_compact_kernel(const int32_t *__restrict__ row_ptr,
                                                                        int32_t num_entities,
                                                                        const int32_t *__restrict__ partials,
                                                                        int32_t *__restrict__ out,
                                                                        int64_t *__restrict__ count_out) {
  __shared__ int2 scratch[kStartWaves];
  const int wave = threadIdx.x / kWave;
  const int64_t v0 = int64_t(blockIdx.x) * kStartTile + int64_t(wave) * kWave * kStartItems;
  const uint32_t f = nonsink_flags(row_ptr, num_entities, v0);
  int before = 0;  // this thread's share of the counts of the blocks before
  for (int64_t b = threadIdx.x; b < int64_t(blockIdx.x); b += kStartThreads) before += partials[b];
  uint64_t m[kStartItems];
  int in_wave = 0;
#pragma unroll
  for (int i = 0; i < kStartItems; ++i) {
    m[i] = __ballot((f >> i) & 1u);
    in_wave += __popcll(m[i]);
  }
  // one sum over the waves: their counts, and the counts of the blocks before
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) before += __shfl_xor(before, off, kWave);
  if (lane_id() == 0) scratch[wave] = make_int2(in_wave, before);
  __syncthreads();
  int64_t at = 0;
  int total = 0;
#pragma unroll
  for (int w = 0; w < kStartWaves; ++w) {
    const int2 s = scratch[w];
    at += s.y + (w < wave ? s.x : 0);
    total += s.x + s.y;
  }
#pragma unroll
  for (int i = 0; i < kStartItems; ++i) {
    if ((f >> i) & 1u) out[at + __popcll(m[i] & lanes_below(lane_id()))] = int32_t(v0 + i * kWave + lane_id());
    at += __popcll(m[i]);
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *count_out = total;
}

}  // namespace

namespace {

// Sizes of the count table of the 4,096-triple tiles and 8-bit digits that the
// workspace size is defined by (callers hold workspaces of that size): the
// passes below fit their tables into it and into free parts of the key buffers.
struct TableSpace {
  size_t counts, partials;
};
TableSpace reserved_tables(int64_t num_triples, int total_bits) {
  int passes = total_bits == 0 ? 1 : int(ceil_div(total_bits, 8));
  if (passes == 3 && total_bits <= 18) passes = 2;
  const int widest = total_bits == 0 ? 1 : int(ceil_div(total_bits, passes));
  const int64_t count_len = (int64_t(1) << widest) * ceil_div(num_triples, 4096);
  return {align_up(size_t(count_len) * 4, 256), align_up(size_t(ceil_div(count_len, kScanTile) + 1) * 4, 256)};
}

int subject_bits(int32_t num_entities) {
  return num_entities > 1 ? 32 - __builtin_clz(uint32_t(num_entities - 1)) : 0;
}

// Table bytes of a pass of `bits`: counts, totals, and the top digit's bases.
size_t table_bytes(int64_t tiles, int bits) {
  return align_up((size_t(1) << bits) * size_t(row_stride(tiles)) * 4, 256) + 2 * align_up(size_t(4) << bits, 256);
}

}  // namespace

SortPlan plan_csr_build(int64_t num_triples, int32_t num_entities) {
  SortPlan p;
  if (num_triples <= 0) return p;
  const int total_bits = subject_bits(num_entities);
  const size_t T = size_t(num_triples);
  const TableSpace space = reserved_tables(num_triples, total_bits);
  size_t off = 0;
  p.off_keys_a = off;  off = align_up(off + T * 4, 256);
  p.off_keys_b = off;  off = align_up(off + T * 4, 256);
  p.off_payload = off; off = align_up(off + T * 8, 256);
  const size_t off_tables = off;
  p.bytes = off + space.counts + space.partials;
  p.total_bits = total_bits;
  if (num_triples <= kMostTile) return p;  // passes == 0: csr_small_kernel
  const int bits = total_bits == 0 ? 1 : total_bits;
  const size_t in_row_ptr = (size_t(num_entities) + 1) * 4;  // less up to 256 bytes of alignment
  // As few passes as digits of at most kMaxDigitBits allow, the bits spread
  // evenly with the odd ones last, or more in the last pass where that brings
  // the bits below it to 16, so that it can write 2-byte keys. Every pass needs
  // room for its table: the reserved one; else, for the first pass, the idle
  // key buffer, for the last one the part of its key buffer that narrow keys
  // leave, for any later one that leaves no bases behind the row_ptr output (the
  // inputs, which that may overlap, have been read by then). Where that
  // is not to be had (some tens of thousands of triples), narrower digits are.
  // Rounds of a tile: as long as the tiles are fewer than about two per CU,
  // smaller tiles use more of the chip (1M triples, scatter of 8 bits: 13.9 us
  // with 8 rounds in 123 tiles).
  const int rounds = num_triples >= (int64_t(4) << 20) ? 8 : num_triples >= (int64_t(2) << 20) ? 4 : 2;
  for (int most = kMaxDigitBits; most > 0; --most)
  for (p.rounds = rounds; p.rounds <= kMostRounds; p.rounds *= 2) {
    p.tiles = ceil_div(num_triples, kSortThreads * p.rounds);
    p.passes = int(ceil_div(bits, most));
    if (p.passes > 4) break;
    const int last = p.passes - 1;
    for (int k = 0; k < p.passes; ++k) p.pass_bits[k] = bits / p.passes + (k >= p.passes - bits % p.passes ? 1 : 0);
    if (p.passes == 3 && bits - p.pass_bits[last] > 16 && bits - 16 <= most) p.pass_bits[last] = bits - 16;
    const int low = bits - p.pass_bits[last];
    if (p.passes == 3) {  // the middle pass has the least room
      p.pass_bits[0] = std::min(most, low - (low - 1) / 2);
      p.pass_bits[1] = low - p.pass_bits[0];
    }
    p.key_out = low == 0 ? 0 : (low <= 16 ? 2 : 4);
    bool fits = true;
    for (int k = 0; k < p.passes; ++k) {
      const size_t need = table_bytes(p.tiles, p.pass_bits[k]);
      const size_t own_keys = align_up(T * size_t(p.key_out), 256);
      const size_t out = k % 2 == 0 ? p.off_keys_a : p.off_keys_b;
      p.table_in_row_ptr[k] = false;
      if (need <= space.counts + space.partials) p.off_tables[k] = off_tables;
      else if (k == 0 && last > 0 && need <= align_up(T * 4, 256)) p.off_tables[k] = p.off_keys_b;
      else if (k == last && need + own_keys <= align_up(T * 4, 256)) p.off_tables[k] = out + own_keys;
      else if (k > 0 && (k < last || p.key_out == 4) && need + 256 <= in_row_ptr) p.table_in_row_ptr[k] = true;
      else fits = false;
    }
    if (fits) return p;
  }
  p.passes = -1;  // cannot happen: for 2 to 8 tiles digits of 7 or 8 bits fit, beyond that wider ones
  return p;
}

namespace {

// What one pass reads and writes.
struct PassArgs {
  const uint32_t *keys_in;
  const int2 *pay_in;
  const int32_t *pred, *obj;  // first pass, instead of pay_in
  void *keys_out;
  int2 *pay_out;
  int64_t n;
  int shift, bits, key_out;
  int32_t *counts, *totals, *bases;
  int64_t tiles;
  int32_t num_entities, num_predicates;
  int32_t *row_ptr;  // first pass: to be marked, or NULL
  int32_t *status;
};

template <bool kFirst, int kRounds, int kKeyOut>
void launch_scatter(const PassArgs &p, hipStream_t stream) {
  const dim3 grid{unsigned(p.tiles)}, block{kSortThreads};
  auto run = [&](auto kernel) {
    kernel<<<grid, block, 0, stream>>>(p.keys_in, p.pay_in, p.pred, p.obj, p.keys_out, p.pay_out, p.n, p.shift, p.bits,
                                       p.counts, p.totals, p.bases, p.tiles, p.num_entities, p.num_predicates, p.status);
  };
  if (p.bits <= 8) run(radix_scatter_kernel<kFirst, kKeyOut, 8, kRounds>);
  else run(radix_scatter_kernel<kFirst, kKeyOut, kMaxDigitBits, kRounds>);
}

template <bool kFirst, int kRounds>
rdf2v_status launch_pass(const PassArgs &p, hipStream_t stream) {
  radix_count_kernel<kFirst, kRounds><<<dim3(unsigned(p.tiles)), dim3(kCountThreads), 0, stream>>>(
      p.keys_in, p.n, p.shift, p.bits, p.num_entities, p.counts, p.tiles, p.row_ptr, p.status);
  RDF2V_LAUNCH_CHECK();
  row_scan_kernel<<<dim3(1u << p.bits), dim3(kScanThreads), 0, stream>>>(p.counts, p.tiles, p.totals);
  RDF2V_LAUNCH_CHECK();
  if (p.key_out == 4) launch_scatter<kFirst, kRounds, 4>(p, stream);
  else if (p.key_out == 2) launch_scatter<kFirst, kRounds, 2>(p, stream);
  else if constexpr (kFirst) launch_scatter<kFirst, kRounds, 0>(p, stream);  // one pass in all
  RDF2V_LAUNCH_CHECK();
  return RDF2V_OK;
}

template <int kRounds>
rdf2v_status launch_pass(bool first, const PassArgs &p, hipStream_t stream) {
  return first ? launch_pass<true, kRounds>(p, stream) : launch_pass<false, kRounds>(p, stream);
}

rdf2v_status launch_row_ptr_fill(int32_t *row_ptr, int32_t num_entities, hipStream_t stream) {
  const int64_t nv = int64_t(num_entities) + 1;
  fill_kernel<<<dim3(unsigned(ceil_div(nv, 256))), dim3(256), 0, stream>>>(row_ptr, nv, -1);
  RDF2V_LAUNCH_CHECK();
  return RDF2V_OK;
}

template <int kKey>
rdf2v_status launch_row_ptr(const SortedKeys &sorted, int64_t T, int32_t num_entities, int32_t *row_ptr,
                            hipStream_t stream) {
  const int gap_run = T < kSparseMax && num_entities >= kSparse * T ? 1 : kGapRun;
  row_ptr_bounds_kernel<kKey><<<dim3(unsigned(ceil_div(T + 1, kBoundThreads * kBoundItems<kKey>))), dim3(kBoundThreads), 0,
                                stream>>>(sorted, T, num_entities, uint32_t(gap_run), row_ptr);
  RDF2V_LAUNCH_CHECK();
  row_ptr_fixup_kernel<kKey><<<dim3(unsigned(ceil_div(int64_t(num_entities) + 1, 256))), dim3(256), 0, stream>>>(
      sorted, T, num_entities, row_ptr);
  RDF2V_LAUNCH_CHECK();
  return RDF2V_OK;
}

}  // namespace

rdf2v_status launch_csr_build(const int32_t *subj, const int32_t *pred, const int32_t *obj,
                              int64_t num_triples, int32_t num_entities, int32_t num_predicates,
                              int32_t *row_ptr_out, int32_t *edges_out, void *workspace,
                              const SortPlan &plan, int32_t *status_dev, hipStream_t stream) {
  const int64_t T = num_triples;
  if (T == 0) {
    const int64_t n = int64_t(num_entities) + 1;
    fill_kernel<<<dim3(unsigned(ceil_div(n, 256))), dim3(256), 0, stream>>>(row_ptr_out, n, 0);
    RDF2V_LAUNCH_CHECK();
    return RDF2V_OK;
  }
  const uint32_t *keys_in = reinterpret_cast<const uint32_t *>(subj);
  int2 *edges2 = reinterpret_cast<int2 *>(edges_out);
  char *ws = static_cast<char *>(workspace);
  if (plan.passes < 0) return RDF2V_ERR_WORKSPACE;
  // row_ptr_out may overlap the inputs (only edges_out may not): it is then left
  // alone until they have been read.
  auto overlaps = [&](const int32_t *in) {
    const uintptr_t a = reinterpret_cast<uintptr_t>(in), b = reinterpret_cast<uintptr_t>(row_ptr_out);
    return a < b + (size_t(num_entities) + 1) * 4 && b < a + size_t(T) * 4;
  };
  bool fill_later = overlaps(subj) || overlaps(pred) || overlaps(obj);
  if (plan.passes == 0) {
    uint32_t *keys = reinterpret_cast<uint32_t *>(ws + plan.off_keys_a);
    const bool with_row_ptr = num_entities <= kSmallEntities && !fill_later;
    csr_small_kernel<<<dim3(1), dim3(kSortThreads), 0, stream>>>(keys_in, pred, obj, int(T), num_entities,
                                                                num_predicates, plan.total_bits,
                                                                with_row_ptr ? row_ptr_out : nullptr, edges2, keys,
                                                                status_dev);
    RDF2V_LAUNCH_CHECK();
    if (with_row_ptr) return RDF2V_OK;
    const rdf2v_status st = launch_row_ptr_fill(row_ptr_out, num_entities, stream);
    if (st != RDF2V_OK) return st;
    return launch_row_ptr<4>({keys, nullptr, 0, 0}, T, num_entities, row_ptr_out, stream);
  }
  int2 *pay_tmp = reinterpret_cast<int2 *>(ws + plan.off_payload);
  // a later pass's table may lie in row_ptr_out until the sort is done
  for (int pass = 0; pass < plan.passes; ++pass) fill_later = fill_later || plan.table_in_row_ptr[pass];
  PassArgs p{};
  p.keys_in = keys_in;
  p.pred = pred;
  p.obj = obj;
  p.n = T;
  p.tiles = plan.tiles;
  p.num_entities = num_entities;
  p.num_predicates = num_predicates;
  for (int pass = 0; pass < plan.passes; ++pass) {
    const bool first = pass == 0, last = pass == plan.passes - 1;
    p.bits = plan.pass_bits[pass];
    p.keys_out = ws + (pass % 2 == 0 ? plan.off_keys_a : plan.off_keys_b);
    p.key_out = last ? plan.key_out : 4;
    // The last pass must land in edges_out, so the payload alternates backwards from it.
    p.pay_out = ((plan.passes - 1 - pass) % 2 == 0) ? edges2 : pay_tmp;
    p.counts = plan.table_in_row_ptr[pass]
                   ? reinterpret_cast<int32_t *>(align_up(reinterpret_cast<uintptr_t>(row_ptr_out), 256))
                   : reinterpret_cast<int32_t *>(ws + plan.off_tables[pass]);
    p.totals = p.counts + align_up((size_t(1) << p.bits) * size_t(row_stride(plan.tiles)) * 4, 256) / 4;
    p.bases = last ? p.totals + align_up(size_t(4) << p.bits, 256) / 4 : nullptr;
    p.row_ptr = first && !fill_later ? row_ptr_out : nullptr;
    p.status = first ? status_dev : nullptr;
    const rdf2v_status st = plan.rounds == 2   ? launch_pass<2>(first, p, stream)
                            : plan.rounds == 4 ? launch_pass<4>(first, p, stream)
                                               : launch_pass<8>(first, p, stream);
    if (st != RDF2V_OK) return st;
    p.keys_in = static_cast<const uint32_t *>(p.keys_out);
    p.pay_in = p.pay_out;
    p.shift += p.bits;
  }
  if (fill_later) {
    const rdf2v_status st = launch_row_ptr_fill(row_ptr_out, num_entities, stream);
    if (st != RDF2V_OK) return st;
  }
  const int top = plan.pass_bits[plan.passes - 1];
  const SortedKeys sorted{p.keys_in, p.bases, 1 << top, p.shift - top};
  if (plan.key_out == 4) return launch_row_ptr<4>(sorted, T, num_entities, row_ptr_out, stream);
  if (plan.key_out == 2) return launch_row_ptr<2>(sorted, T, num_entities, row_ptr_out, stream);
  return launch_row_ptr<0>(sorted, T, num_entities, row_ptr_out, stream);
}

size_t nonsink_workspace_bytes(int32_t num_entities) {
  const int64_t nb = ceil_div(int64_t(num_entities > 0 ? num_entities : 0), kScanTile);
  return align_up(size_t(nb + 1) * 4, 256);
}

rdf2v_status launch_nonsink_starts(const int32_t *row_ptr, int32_t num_entities, int32_t *starts_out,
                                   int64_t *count_out, void *workspace, hipStream_t stream) {
  // no entities: one block that finds none and writes the count
  const int64_t nb = num_entities > 0 ? ceil_div(int64_t(num_entities), kStartTile) : 1;
  int32_t *partials = static_cast<int32_t *>(workspace);
  if (nb > 1) {
    nonsink_count_kernel<<<dim3(unsigned(nb)), dim3(kStartThreads), 0, stream>>>(row_ptr, num_entities, partials);
    RDF2V_LAUNCH_CHECK();
  }
  nonsink_compact_kernel<<<dim3(unsigned(nb)), dim3(kStartThreads), 0, stream>>>(row_ptr, num_entities, partials,
                                                                                starts_out, count_out);
  RDF2V_LAUNCH_CHECK();
  return RDF2V_OK;
}

}  // namespace rdf2v
