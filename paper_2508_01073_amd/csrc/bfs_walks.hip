// BFS walks on gfx950 (gpuRDF2vec Sec. 3.1): per root, a depth-limited BFS
// tree in which every reached entity has one predecessor, and one walk per
// leaf, root to leaf.
//
// The tree is the one a queue-order BFS builds: the entities of a level are
// expanded in the order they were reached, each through its out-edge records in
// CSR order, and an entity gets as parent the first (entity, record) that
// reaches it. The kernels get the same tree level-synchronously:
//   * the (entity, record) pairs of a level are numbered q = 0, 1, ... in
//     exactly that order (a block scan of the level's degrees);
//   * every pair that reaches an entity not yet in the tree offers q to that
//     entity with an atomic minimum, so the smallest q wins;
//   * the winners, in q order (a block scan), are the next level.
// Leaves are then ranked in the order reached and the first max_walks become
// rows root, V+p_1, v_1, ..., leaf.
//
// Three LDS tiers run a root in one workgroup with all its state in LDS: the
// tree above the depth limit, the level's degree prefix and an open-addressing
// hash table of the entities reached so far (tree members and this level's
// offers). Every root starts in one tier, picked from the expected tree size; a
// root whose tree outgrows a tier is abandoned there and queued for the next.
// The last pass, a persistent grid of workgroups that each own a slice of the
// workspace, reruns the roots no tier could hold from scratch: it takes the
// pairs of a level in order, a chunk at a time, with one "reached" bit per
// entity instead of per-entity offers. All loops are bounded by the tree and
// level sizes or the table size; a workgroup never waits for another. The
// entities of a level are distinct, so in a consistent CSR their rows hold at
// most num_edges records; a level of more (rows that overlap, each of them in
// range) ends its root with RDF2V_STATUS_BAD_CSR, so that the pair numbers of
// every level that is walked are exact in 31 bits and increase.

#include <algorithm>

#include "common.hpp"
#include "launch.hpp"

namespace rdf2v {
namespace {

struct BfsArgs {
  const int32_t *row_ptr;
  const int32_t *edges;  // (predicate, object) pairs
  const int32_t *roots;
  int32_t *tokens;
  int32_t *lens;
  int32_t *counts;
  int32_t *status;
  int32_t *queue_counts;  // [kQueueCounters]: lengths of the queues below, then how far each has been taken
  int32_t *queue[3];      // roots (indices into roots) LDS tier i could not hold
  int64_t num_roots;
  int64_t num_edges;
  int32_t num_entities;
  int32_t num_predicates;
  int32_t depth;
  int32_t max_walks;
};

// Slots of queue_counts: the lengths of the three tiers' queues, then how far
// each was taken (tier t takes queue t - 1 through slot 3 + t: slots 4 and 5),
// then the bitmap pass: queue 2 taken, and the length and taken count of the
// queue of its second run (queue 0 again, which is used up by then).
constexpr int kQueueCounters = 9;
constexpr int kWideTaken = 6, kWide2Length = 7, kWide2Taken = 8;

// The workspace is sized in units of 36 bytes per entity, about 4 GiB of them
// at most and one at least.
inline size_t slice_bytes(int64_t V) {
  return align_up(size_t(V) * 4, 256) * 6 + align_up(size_t(V) * 8, 256) + align_up(size_t(V + 1) * 4, 256);
}

// Workspace: the queue counters, three queues (one int32 per root each), the
// slices of the bitmap pass.
inline size_t queue_bytes(int64_t num_roots) { return 256 + 3 * align_up(size_t(num_roots) * 4, 256); }

// ---------------------------------------------------------------------------
// LDS tiers: one root at a time per workgroup, all state in LDS.

// Three LDS tiers of growing capacity and LDS footprint: one wave per root
// (about 6.3 KB of LDS, 24 workgroups per CU), 256 threads (about 25 KB, 6
// per CU) and 512 threads (about 50 KB, 3 per CU). A root goes to the next
// tier when it outgrows one. All keep VGPRs <= 80 for six waves per SIMD (the
// big tier spills a few registers for its four rounds).
struct TinyTier {
  static constexpr int kThreads = 64;
  static constexpr int kRounds = 2;
  static constexpr int kLog = 9;
  static constexpr int kCap = 384;
  static constexpr int kTreeCap = 96;
  static constexpr int kWavesPerSimd = 6;
};
struct SmallTier {
  static constexpr int kThreads = 256;
  static constexpr int kRounds = 2;     // rounds of kThreads pairs whose records are loaded together
  static constexpr int kLog = 11;       // hash table of 2^kLog slots
  static constexpr int kCap = 1536;     // most entities a root may reach here
  static constexpr int kTreeCap = 384;  // most of them above the depth limit (kept as tree nodes)
  static constexpr int kWavesPerSimd = 6;
  static constexpr int kPerCu = 6;
};
struct BigTier {
  static constexpr int kThreads = 512;
  static constexpr int kRounds = 4;
  static constexpr int kLog = 12;
  static constexpr int kCap = 3072;
  static constexpr int kTreeCap = 768;
  static constexpr int kWavesPerSimd = 6;
  static constexpr int kPerCu = 3;
};
// A level of more than kGiveUp * kCap pairs leaves a tier before its offers
// (1,000 roots of the 20M-triple power-law graph that no tier can hold: the
// two tiers took 2.8 + 8.1 ms until their tables were full, 0.06 + 0.09 ms
// with this and the checks while a table fills). At 2, 4, 8 and 16, in us:
//   power law, 50K entities, 300K triples, depth 2, 20,000 roots: 1,149, 1,307, 1,390, 1,457
//   power law, 10K, 60K, depth 3, 5,000 roots:                      928,   940, 1,016, 1,068
//   power law, 200K, 2M, depth 2, 2,000 roots:                      795,   803,   787,   799
//   uniform, 100K, 2M, depth 3, 2,000 roots:                        620,   772,   766,   774
//   4,000 roots with 7,000 pairs to 2,500 entities at depth 2:      499,   232,   233,   231
//   the same with 24,000 pairs:                                     690,   692,   548,   544
// So 2 serves graphs whose levels grow with their pairs, and levels of 6,000 to
// 24,000 pairs that meet few entities pay up to twice for it. (Leaving instead
// when the first chunk of such a level repeats too little took 239 in the fifth
// row, but 2.4 % more for the 1M-triple uniform graph, which never gets there,
// through the registers it holds, and up to 55 % more for some hundred roots
// of small power-law graphs, whose levels look like few entities at first.)
constexpr int32_t kGiveUp = 2;
constexpr int32_t kFreeSlot = -1;
constexpr uint32_t kNoOffer = 0xFFFFFFFFu;

// Fibonacci hashing of an entity id to one of 2^kLog slots.
template <int kLog>
__device__ __forceinline__ int32_t entity_slot(int32_t x) {
  return int32_t((uint32_t(x) * 0x9E3779B1u) >> (32 - kLog));
}

__device__ __forceinline__ int32_t wave_sum(int32_t v) {
  return __builtin_amdgcn_readlane(wave_inclusive_sum(v), kWave - 1);
}

__device__ __forceinline__ int32_t wave_index() { return __builtin_amdgcn_readfirstlane(int32_t(threadIdx.x) / kWave); }

// Set bits of a wave-wide mask below the calling lane.
__device__ __forceinline__ int32_t lanes_below(uint64_t b) {
  return int32_t(__builtin_amdgcn_mbcnt_hi(uint32_t(b >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(b), 0u)));
}

// Exclusive prefix sum over the block (one value per thread) and its total.
// One barrier; scratch holds NT/64 ints and must not be written again before
// the next barrier (callers alternate between two scratch buffers).
template <int NT>
__device__ __forceinline__ int32_t block_scan(int32_t x, int32_t *scratch, int32_t &total) {
  constexpr int W = NT / kWave;
  const int32_t inc = wave_inclusive_sum(x);
  if constexpr (W == 1) {
    total = __builtin_amdgcn_readlane(inc, kWave - 1);
    return inc - x;
  } else {
    const int lane = lane_id();
    const int32_t w = wave_index();
    if (lane == kWave - 1) scratch[w] = inc;
    __syncthreads();
    const int32_t waves = wave_inclusive_sum(lane < W ? scratch[lane] : 0);
    total = __builtin_amdgcn_readlane(waves, W - 1);
    return (w > 0 ? __builtin_amdgcn_readlane(waves, w - 1) : 0) + inc - x;
  }
}

// Ranks, in pair order, the flagged pairs of a chunk whose round k holds pair
// c0 + k*NT + threadIdx.x: rank[k] counts the flagged pairs before it in the
// chunk; `total` is their number. One barrier; cnt_s holds R * NT/64 ints and
// is reused like the scratch of block_scan.
template <int NT, int R>
__device__ __forceinline__ void rank_chunk(uint32_t mask, int32_t (&rank)[R], int32_t &total, int32_t *cnt_s) {
  constexpr int W = NT / kWave;
  static_assert(R * W <= kWave, "one count per lane");
  const int lane = lane_id();
  const int32_t w = wave_index();
  uint64_t b[R];
#pragma unroll
  for (int k = 0; k < R; ++k) b[k] = __ballot((mask >> k) & 1u);
  // counts in pair order: round-major, then wave
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < R; ++k) cnt_s[k * W + w] = __popcll(b[k]);
  }
  __syncthreads();
  const int32_t inc = wave_inclusive_sum(lane < R * W ? cnt_s[lane] : 0);
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int32_t idx = k * W + w;
    rank[k] = (idx > 0 ? __builtin_amdgcn_readlane(inc, idx - 1) : 0) + lanes_below(b[k]);
  }
  total = __builtin_amdgcn_readlane(inc, R * W - 1);
}

// Table entries: key = entity, value = 0 for a tree member, else 1 + the
// smallest pair index of the current level that reached it. Every entity
// inserted during a level's offers has a winning pair, so after the level the
// entry count is the tree size.
//
// Entities at the depth limit are leaves: they are not stored as tree nodes.
// Their pairs are walked twice more instead, once to mark which nodes of the
// level above get a child, and once, after the stored leaves are ranked, to
// write their walks in pair order.
//
// The pairs of a level are taken in chunks of R rounds of NT consecutive
// pairs; a thread loads the records of its R pairs together. A level of at
// most one chunk keeps its records (and winners) in registers for all its
// passes.
//
// Without in_queue, workgroup b takes roots b, b + G, ...; with it, the
// workgroups take its in_count entries one at a time through the counter
// `taken`. Roots the tier cannot hold are appended to out_queue.
template <int NT, int R, int kLog, int kCap, int kTreeCap, int kWpe>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(kWpe))) void bfs_lds_kernel(
    const BfsArgs a, const int32_t *in_queue, const int32_t *in_count, int32_t *taken, int32_t *out_queue,
    int32_t *out_count) {
  constexpr int kSlots = 1 << kLog;
  constexpr int32_t kChunk = NT * R;
  static_assert(kCap < kSlots && kTreeCap <= kCap && kTreeCap <= 32767, "table and tree sizes");
  static_assert(kSlots % (4 * NT) == 0, "the table is cleared four slots per thread at a time");
  static_assert(R <= 32, "win masks are 32-bit");
  // Degrees are capped one above kLongRow, so that those of a level add up to
  // about 2^30 at most whatever row_ptr holds.
  constexpr int32_t kLongRow = (1 << 30) / kTreeCap;
  __shared__ int32_t scan_scratch[2][R * (NT / kWave)];  // alternated between block-wide scans
  __shared__ __align__(16) int32_t h_key[kSlots];
  __shared__ __align__(16) uint32_t h_val[kSlots];
  __shared__ int32_t t_ent[kTreeCap];
  __shared__ int32_t t_pred[kTreeCap];
  __shared__ int16_t t_par[kTreeCap];
  __shared__ uint8_t t_lev[kTreeCap];
  __shared__ uint8_t t_child[kTreeCap];
  __shared__ int32_t t_lo[kTreeCap];        // CSR row start of each tree node
  __shared__ int32_t t_deg[kTreeCap];       // and its out-degree (0 for a bad row)
  __shared__ int32_t dpre_s[kTreeCap + 1];  // degree prefix of the level being expanded
  __shared__ int32_t used_s;                // table entries
  __shared__ int32_t overflow_s;
  __shared__ int32_t next_s;
  const int t = threadIdx.x;
  const int32_t V = a.num_entities;
  const uint32_t E = uint32_t(a.num_edges);
  const int64_t width = 2 * int64_t(a.depth) + 1;
  const int2 *edges = reinterpret_cast<const int2 *>(a.edges);

  // Slot of x, inserting it if absent (then `inserted` is incremented); -1
  // when the table is full (the root is then left to the next tier). The
  // entry count is checked against kCap once all offers of a level are in.
  auto claim = [&](int32_t x, int32_t &inserted) -> int32_t {
    int32_t s = entity_slot<kLog>(x);
    for (int n = 0; n < kSlots; ++n) {
      const int32_t k = __hip_atomic_load(h_key + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (k == x) return s;
      if (k == kFreeSlot) {
        const int32_t old = atomicCAS(h_key + s, kFreeSlot, x);
        if (old == kFreeSlot) {
          ++inserted;
          return s;
        }
        if (old == x) return s;
      }
      s = (s + 1) & (kSlots - 1);
    }
    overflow_s = 1;
    return -1;
  };
  auto find = [&](int32_t x) -> int32_t {
    int32_t s = entity_slot<kLog>(x);
    for (int n = 0; n < kSlots; ++n) {
      const int32_t k = h_key[s];
      if (k == x) return s;
      if (k == kFreeSlot) break;
      s = (s + 1) & (kSlots - 1);
    }
    return -1;
  };

  // A level of more pairs leaves the tier at once: many more than the table
  // holds entities outgrow it (nearly always: only repeats could keep them in),
  // a capped degree may be among more than kLongRow, and more than the CSR has
  // records come from overlapping rows, which the bitmap pass reports.
  const int32_t most_pairs = min(V > kCap ? kGiveUp * kCap : kLongRow, int32_t(E));

  int flags = 0;
  int32_t phase = 0;
  auto scratch = [&]() -> int32_t * { return scan_scratch[phase ^= 1]; };
  const int64_t n_in = in_queue != nullptr ? int64_t(*in_count) : a.num_roots;
  if (int64_t(blockIdx.x) >= n_in) return;  // uniform; an empty queue costs one load per workgroup
  for (int64_t k_in = blockIdx.x;; k_in += gridDim.x) {
    if (in_queue != nullptr) {  // uniform
      if (t == 0) next_s = atomicAdd(taken, 1);
      __syncthreads();
      k_in = uint32_t(next_s);  // past the queue's end by the grid at most
      __syncthreads();
    }
    if (k_in >= n_in) break;
    const int64_t r = in_queue != nullptr ? int64_t(in_queue[k_in]) : k_in;
    const int32_t root = a.roots[r];
    if (uint32_t(root) >= uint32_t(V)) {
      if (t == 0) a.counts[r] = 0;
      flags |= RDF2V_STATUS_ID_OUT_OF_RANGE;
      continue;  // uniform: every lane skips the same root
    }
    for (int i = t; i < kSlots / 4; i += NT) {
      reinterpret_cast<int4 *>(h_key)[i] = make_int4(kFreeSlot, kFreeSlot, kFreeSlot, kFreeSlot);
      reinterpret_cast<uint4 *>(h_val)[i] = make_uint4(kNoOffer, kNoOffer, kNoOffer, kNoOffer);
    }
    __syncthreads();
    if (t == 0) {
      const int32_t lo = a.row_ptr[root], hi = a.row_ptr[root + 1];
      const bool ok = uint32_t(lo) <= uint32_t(hi) && uint32_t(hi) <= E;
      if (!ok) flags |= RDF2V_STATUS_BAD_CSR;
      t_lo[0] = lo;
      t_deg[0] = ok ? min(hi - lo, kLongRow + 1) : 0;
      const int32_t s0 = entity_slot<kLog>(root);
      h_key[s0] = root;
      h_val[s0] = 0;
      used_s = 1;
      overflow_s = 0;
      t_ent[0] = root;
      t_pred[0] = -1;
      t_par[0] = -1;
      t_lev[0] = 0;
      t_child[0] = 0;
    }
    __syncthreads();
    int32_t lb = 0, le = 1;      // the level being expanded: tree nodes [lb, le)
    int32_t nlev = 0, total = 0;  // its size and its number of (entity, record) pairs
    int32_t last_wins = 0;       // entities reached at the depth limit
    bool overflow = false;
    // The thread's pairs of the chunk at c0 (round k: pair c0 + k*NT + t): level
    // entity index (-1 past the end), record, and table slot of the record's
    // entity (-1 if none).
    int32_t node_k[R];
    int2 rec_k[R];
    int32_t slot_k[R];
    auto load_chunk = [&](int32_t c0) {
#pragma unroll
      for (int k = 0; k < R; ++k) {
        node_k[k] = -1;
        rec_k[k] = make_int2(0, -1);
      }
      if (c0 + wave_index() * kWave >= total) return;  // uniform: no pair of this wave in the chunk
      // largest i with dpre[i] <= q, by halving steps from the top bit of nlev
      int32_t lo[R];
#pragma unroll
      for (int k = 0; k < R; ++k) lo[k] = 0;
      for (int32_t step = int32_t(1u << (31 - __builtin_clz(uint32_t(nlev)))); step > 0; step >>= 1) {
#pragma unroll
        for (int k = 0; k < R; ++k) {
          const int32_t m = lo[k] + step;
          if (m < nlev && dpre_s[m] <= c0 + k * NT + t) lo[k] = m;
        }
      }
#pragma unroll
      for (int k = 0; k < R; ++k) {
        const int32_t q = c0 + k * NT + t;
        node_k[k] = q < total ? lo[k] : -1;
        rec_k[k] = q < total ? edges[uint32_t(t_lo[lb + lo[k]] + (q - dpre_s[lo[k]]))] : make_int2(0, -1);
      }
    };
    // Bit k set: the thread's round-k pair reaches its entity first. With
    // `known`, slot_k holds the slots from this chunk's offers; else they are
    // looked up.
    auto winners = [&](int32_t c0, bool known) -> uint32_t {
      uint32_t m = 0;
#pragma unroll
      for (int k = 0; k < R; ++k) {
        if (!known) slot_k[k] = node_k[k] >= 0 && uint32_t(rec_k[k].y) < uint32_t(V) ? find(rec_k[k].y) : -1;
        if (slot_k[k] >= 0 && h_val[slot_k[k]] == uint32_t(c0 + k * NT + t) + 1u) m |= 1u << k;
      }
      return m;
    };
    uint32_t last_mask = 0;  // winners of a one-chunk last level
    for (int32_t lev = 0; lev < a.depth && lb < le; ++lev) {
      nlev = le - lb;  // le <= kTreeCap
      // Degree prefix of the level (rows were read when its nodes were added).
      int32_t carry = 0;
      for (int32_t c0 = lb; c0 < le; c0 += NT) {
        const int32_t i = c0 + t;
        int32_t tot;
        const int32_t ex = block_scan<NT>(i < le ? t_deg[i] : 0, scratch(), tot);
        if (i < le) dpre_s[i - lb] = carry + ex;
        carry += tot;
      }
      total = carry;
      if (t == 0) dpre_s[nlev] = total;
      __syncthreads();
      if (total > most_pairs) {  // uniform
        overflow = true;
        break;
      }
      const bool one_chunk = total <= kChunk;  // uniform: records stay in registers
      const bool last = lev + 1 == a.depth;
      // Offers (tree members hold 0 and ignore them).
      // Where the level can outgrow the tier, a wave adds what it inserted after
      // every round and stops once the capacity is passed: the table never
      // comes near full, where every further offer would probe most of it.
      bool full = false;
      int32_t inserted = 0;
      const int32_t cap = last ? kCap : kTreeCap;
      const bool may_outgrow = used_s + total > cap;  // uniform: no wave adds before the barrier below otherwise
      for (int32_t c0 = 0; c0 < total && (!may_outgrow || __ballot(full) == 0); c0 += kChunk) {
        load_chunk(c0);
#pragma unroll
        for (int k = 0; k < R; ++k) {
          slot_k[k] = -1;
          if (may_outgrow && (k > 0 || c0 > 0)) {
            const int32_t sum = wave_sum(inserted);
            inserted = 0;
            if (lane_id() == 0 && sum > 0) atomicAdd(&used_s, sum);
            const int32_t used = __hip_atomic_load(&used_s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            full = __ballot(full || used > cap) != 0;  // the whole wave stops, so the wave sums stay whole
          }
          if (full || node_k[k] < 0) continue;
          const int32_t x = rec_k[k].y;
          if (uint32_t(x) >= uint32_t(V)) {
            flags |= RDF2V_STATUS_ID_OUT_OF_RANGE;
            continue;
          }
          const int32_t s = claim(x, inserted);
          if (s < 0) {
            full = true;
          } else {
            slot_k[k] = s;
            atomicMin(h_val + s, uint32_t(c0 + k * NT + t) + 1u);
          }
        }
      }
      inserted = wave_sum(inserted);
      if (lane_id() == 0 && inserted > 0) atomicAdd(&used_s, inserted);
      __syncthreads();
      if (overflow_s || used_s > cap) {  // uniform
        overflow = true;
        break;
      }
      if (last) {
        // Nodes of this level with a winning pair are not leaves.
        int32_t n_wins = 0;
        for (int32_t c0 = 0; c0 < total; c0 += kChunk) {
          if (!one_chunk) load_chunk(c0);
          const uint32_t m = winners(c0, one_chunk);
#pragma unroll
          for (int k = 0; k < R; ++k)
            if (m & (1u << k)) t_child[lb + node_k[k]] = 1;
          n_wins += __popc(m);
          last_mask = m;
        }
        {
          int32_t all;
          (void)block_scan<NT>(n_wins, scratch(), all);
          last_wins = all;
        }
        break;  // lb, le, nlev, total (and a one-chunk level's records) stay for the rows
      }
      // Winners in pair order become the next level.
      int32_t added = 0;
      for (int32_t c0 = 0; c0 < total; c0 += kChunk) {
        if (!one_chunk) load_chunk(c0);
        int32_t rank[R], tot, row_lo_k[R], row_hi_k[R];
        const uint32_t m = winners(c0, one_chunk);
#pragma unroll
        for (int k = 0; k < R; ++k) {  // the new nodes' rows, in flight across the ranking
          row_lo_k[k] = row_hi_k[k] = 0;
          if (m & (1u << k)) {
            row_lo_k[k] = a.row_ptr[rec_k[k].y];
            row_hi_k[k] = a.row_ptr[rec_k[k].y + 1];
          }
        }
        rank_chunk<NT, R>(m, rank, tot, scratch());
#pragma unroll
        for (int k = 0; k < R; ++k) {
          if (m & (1u << k)) {
            const int32_t pos = le + added + rank[k];  // < used_s <= kTreeCap
            const int32_t node = lb + node_k[k];
            const bool ok = uint32_t(row_lo_k[k]) <= uint32_t(row_hi_k[k]) && uint32_t(row_hi_k[k]) <= E;
            if (!ok) flags |= RDF2V_STATUS_BAD_CSR;
            t_ent[pos] = rec_k[k].y;
            t_pred[pos] = rec_k[k].x;
            t_par[pos] = int16_t(node);
            t_lev[pos] = uint8_t(lev + 1);
            t_child[pos] = 0;
            t_lo[pos] = row_lo_k[k];
            t_deg[pos] = ok ? min(row_hi_k[k] - row_lo_k[k], kLongRow + 1) : 0;
            t_child[node] = 1;
            h_val[slot_k[k]] = 0;
          }
        }
        added += tot;
      }
      lb = le;
      le += added;
      __syncthreads();
    }
    if (overflow) {
      if (t == 0) {
        // a level that even the last tier would give up goes to the bitmap pass
        const bool skip = V > BigTier::kCap && total > kGiveUp * BigTier::kCap;
        int32_t *q = skip ? a.queue[2] : out_queue;
        q[atomicAdd(skip ? a.queue_counts + 2 : out_count, 1)] = int32_t(r);
      }
      continue;  // the clearing loop of the next root starts after this root's last barrier
    }
    // Walk rows: root, then the tokens of `node` and its ancestors up to level h.
    auto write_path = [&](int32_t *row, int32_t node, int32_t h) {
      for (int32_t step = h; step >= 1; --step) {
        row[2 * step] = t_ent[node];
        row[2 * step - 1] = V + t_pred[node];
        node = t_par[node];
      }
      row[0] = root;
    };
    // Leaves in the order reached, the stored tree nodes first: the first
    // max_walks become walks.
    int32_t leaves = 0;
    for (int32_t c0 = 0; c0 < le; c0 += NT) {
      const int32_t i = c0 + t;
      const int32_t leaf = i < le ? int32_t(t_child[i] == 0) : 0;
      int32_t tot;
      const int32_t ex = block_scan<NT>(leaf, scratch(), tot);
      const int32_t idx = leaves + ex;
      if (leaf && idx < a.max_walks) {
        const int32_t h = t_lev[i];
        int32_t *row = a.tokens + (r * a.max_walks + idx) * width;
        write_path(row, i, h);
        for (int64_t j = 2 * int64_t(h) + 1; j < width; ++j) row[j] = -1;
        a.lens[r * a.max_walks + idx] = 2 * h + 1;
      }
      leaves += tot;
    }
    // Then the entities at the depth limit, in pair order.
    if (last_wins > 0 && leaves < a.max_walks) {
      const bool one_chunk = total <= kChunk;
      int32_t added = 0;
      for (int32_t c0 = 0; c0 < total; c0 += kChunk) {
        uint32_t m = last_mask;
        if (!one_chunk) {
          load_chunk(c0);
          m = winners(c0, false);
        }
        int32_t rank[R], tot;
        rank_chunk<NT, R>(m, rank, tot, scratch());
#pragma unroll
        for (int k = 0; k < R; ++k) {
          const int32_t idx = leaves + added + rank[k];
          if ((m & (1u << k)) && idx < a.max_walks) {
            int32_t *row = a.tokens + (r * a.max_walks + idx) * width;
            row[2 * a.depth] = rec_k[k].y;
            row[2 * a.depth - 1] = V + rec_k[k].x;
            write_path(row, lb + node_k[k], a.depth - 1);
            a.lens[r * a.max_walks + idx] = int32_t(width);
          }
        }
        added += tot;
        if (leaves + added >= a.max_walks) break;  // uniform
      }
    }
    leaves += last_wins;
    if (t == 0) {
      a.counts[r] = min(leaves, a.max_walks);
      if (leaves > a.max_walks) flags |= RDF2V_STATUS_CAPACITY;
    }
    __syncthreads();  // the LDS is reused by the next root
  }
  if (flags && a.status != nullptr) atomicOr(a.status, flags);
}

__global__ void bfs_queue_reset_kernel(int32_t *queue_counts) {
  if (threadIdx.x < kQueueCounters) queue_counts[threadIdx.x] = 0;
}

// ---------------------------------------------------------------------------
// Bitmap pass: the roots no tier could hold (in a power-law graph nearly every
// root that reaches a hub: levels of 10^5 to 10^7 pairs).
//
// One workgroup runs a root and takes a level's pairs in order, kWideChunk at
// a time, so "reached before this chunk" is one bit per entity and an entity
// belongs to the first pair that reaches it without any per-entity offers:
//   * filter: every thread loads kWideRounds records and tests their bits; on a
//     hub's row, where almost all pairs meet entities already reached, a chunk
//     ends here;
//   * the candidates left are numbered in pair order and settled kWideThreads
//     at a time: equal entities meet in an LDS table that keeps the first,
//     which becomes a node, sets its bit and marks its parent.
// What bounds it is the latency of a chunk (records, bits, one to five
// barriers), so the bitmap lives in LDS while it fits (V up to about 1.07M
// entities; the random bit tests and updates then never leave the CU) and in
// the workgroup's slice otherwise, and a chunk is as wide as registers allow.
// Measured on the 20M-triple power-law graph (1M entities, depth 2, 1,000
// roots of 290K pairs on average and 5M at most): 2.4 ms, calls of 2.4 to 3.4 ms
// by the roots drawn: the time of the root with most pairs, against 165 ms with
// 64-bit offers per entity in the workspace (two random accesses at agent scope
// per pair, 119 workgroups).
// A slice holds 25 bytes per tree node: entity, parent, predicate, a
// has-a-child byte, and for the nodes of the level being expanded that have
// records their position, row start and degree prefix.
// At the depth limit only the first max_walks nodes are kept (nothing else of
// them is ever needed). A root with more nodes than a slice holds is queued
// for a second run of the same kernel with fewer, V-sized slices.
constexpr int kWideThreads = 1024;
constexpr int kWideRounds = 8;
constexpr int32_t kWideChunk = kWideThreads * kWideRounds;
constexpr int kWideWindow = 1024;  // nodes of a level whose rows and prefix are in LDS at a time
constexpr int kWideSlots = 2 * kWideThreads;
constexpr int kWideStreamRow = kWideChunk / 2;  // shortest (rest of a) row that is streamed on its own

// Static LDS of the kernel below, rounded up: what a bitmap in LDS leaves it.
constexpr size_t kWideStaticLds = 32 << 10;

struct WidePass {
  const int32_t *in_queue;
  const int32_t *in_count;
  int32_t *taken;
  int32_t *out_queue;  // roots with more than node_cap nodes (none when node_cap >= V)
  int32_t *out_count;
  char *slices;
  size_t slice_bytes;
  int32_t node_cap;
};

inline size_t wide_bitmap_bytes(int64_t V) { return align_up(size_t((V + 31) / 32) * 4, 256); }
// Bytes of a slice of `cap` nodes, and how many nodes a slice of `bytes` holds.
inline size_t wide_slice_bytes(int64_t cap) { return 6 * align_up(size_t(cap) * 4, 256) + align_up(size_t(cap), 256); }
inline int64_t wide_slice_nodes(size_t bytes) { return bytes < 8192 ? 0 : int64_t((bytes - 7 * 256) / 25); }

// Ranks, in pair order, the flagged pairs of a chunk whose wave w holds 64 R
// consecutive pairs, 64 per round (as rank_chunk otherwise; 128 (wave, round)
// counts, two per lane). One barrier; cnt_s must not be
// written again before the next one.
template <int NT, int R>
__device__ __forceinline__ void rank_wide_chunk(uint32_t mask, int32_t (&rank)[R], int32_t &total, int32_t *cnt_s) {
  constexpr int W = NT / kWave;
  static_assert(R * W == 2 * kWave, "two counts per lane");
  const int lane = lane_id();
  const int32_t w = wave_index();
  uint64_t b[R];
#pragma unroll
  for (int k = 0; k < R; ++k) b[k] = __ballot((mask >> k) & 1u);
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < R; ++k) cnt_s[w * R + k] = __popcll(b[k]);
  }
  __syncthreads();
  const int32_t c0 = cnt_s[2 * lane], c1 = cnt_s[2 * lane + 1];
  const int32_t inc = wave_inclusive_sum(c0 + c1);
  const int32_t ex0 = inc - c0 - c1, ex1 = inc - c1;  // counts before entries 2*lane and 2*lane + 1
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int32_t idx = w * R + k;
    const int32_t before = (idx & 1) ? __builtin_amdgcn_readlane(ex1, idx >> 1) : __builtin_amdgcn_readlane(ex0, idx >> 1);
    rank[k] = before + lanes_below(b[k]);
  }
  total = __builtin_amdgcn_readlane(inc, kWave - 1);
}

template <bool kLdsBits>
__global__ __launch_bounds__(kWideThreads) void bfs_wide_kernel(const BfsArgs a, const WidePass p) {
  constexpr int NT = kWideThreads, R = kWideRounds;
  extern __shared__ __align__(16) uint32_t lds_bits[];  // kLdsBits: one bit per entity
  __shared__ int32_t scan_scratch[2][2 * kWave];        // alternated between block-wide scans
  __shared__ uint32_t win_pre[kWideWindow + kWave];  // past the window's nodes: above any pair's number
  __shared__ int32_t win_lo[kWideWindow];
  __shared__ uint8_t win_child[kWideWindow];
  __shared__ int32_t c_ent[NT], c_pred[NT], c_node[NT];  // the candidates being settled
  __shared__ uint32_t table[kWideSlots];                 // 1 + the first candidate of an entity, 0 if free
  __shared__ int32_t level_begin[RDF2V_MAX_DEPTH + 2];
  __shared__ int32_t next_s;
  const int t = threadIdx.x;
  const int32_t V = a.num_entities;
  const uint32_t E = uint32_t(a.num_edges);
  const int64_t width = 2 * int64_t(a.depth) + 1;
  const int2 *edges = reinterpret_cast<const int2 *>(a.edges);

  const int32_t n_in = *p.in_count;
  if (int32_t(blockIdx.x) >= n_in) return;  // uniform; an empty queue costs one load per workgroup
  char *slice = p.slices + size_t(blockIdx.x) * p.slice_bytes;
  const int64_t bit_words = (int64_t(V) + 31) / 32;
  uint32_t *bits = lds_bits;
  if (!kLdsBits) {
    bits = reinterpret_cast<uint32_t *>(slice);
    slice += align_up(size_t(bit_words) * 4, 256);
  }
  const size_t a4 = align_up(size_t(p.node_cap) * 4, 256);
  int32_t *ent = reinterpret_cast<int32_t *>(slice);
  int32_t *parent = reinterpret_cast<int32_t *>(slice + a4);
  int32_t *pred = reinterpret_cast<int32_t *>(slice + 2 * a4);
  // of the level being expanded, for its nodes with records: position, row start, degree prefix
  int32_t *x_node = reinterpret_cast<int32_t *>(slice + 3 * a4);
  int32_t *x_lo = reinterpret_cast<int32_t *>(slice + 4 * a4);
  int32_t *x_pre = reinterpret_cast<int32_t *>(slice + 5 * a4);
  uint8_t *has_child = reinterpret_cast<uint8_t *>(slice + 6 * a4);

  auto visited = [&](int32_t x) -> bool {
    const uint32_t w = kLdsBits ? bits[uint32_t(x) >> 5]
                                : __hip_atomic_load(bits + (uint32_t(x) >> 5), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return (w >> (x & 31)) & 1u;
  };
  auto visit = [&](int32_t x) { atomicOr(bits + (uint32_t(x) >> 5), 1u << (x & 31)); };

  int flags = 0;
  int32_t phase = 0;
  auto scratch = [&]() -> int32_t * { return scan_scratch[phase ^= 1]; };
  for (;;) {
    if (t == 0) next_s = atomicAdd(p.taken, 1);
    __syncthreads();
    const uint32_t k_in = uint32_t(next_s);  // past the queue's end by the grid at most
    __syncthreads();
    if (k_in >= uint32_t(n_in)) break;
    const int64_t r = p.in_queue[k_in];
    const int32_t root = a.roots[r];  // in range: the tiers queue no other
    if constexpr (kLdsBits) {
      for (int64_t i = t; i < (bit_words + 3) / 4; i += NT) reinterpret_cast<uint4 *>(bits)[i] = make_uint4(0, 0, 0, 0);
    } else {
      for (int64_t i = t; i < bit_words; i += NT)
        __hip_atomic_store(bits + i, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (t == 0) {
      visit(root);
      ent[0] = root;
      parent[0] = -1;
      pred[0] = -1;
      has_child[0] = 0;
      level_begin[0] = 0;
      level_begin[1] = 1;
    }
    __syncthreads();
    int32_t lb = 0, le = 1;   // the level being expanded: nodes [lb, le)
    int32_t levels = 1;       // levels with stored begins: level l is [level_begin[l], level_begin[l + 1])
    int32_t last_wins = 0;    // entities reached at the depth limit, or any number above max_walks (stored from le on)
    bool overflow = false, overlap = false;
    for (int32_t lev = 0; lev < a.depth && lb < le && !overflow; ++lev) {
      const int32_t nlev = le - lb;
      const bool last = lev + 1 == a.depth;
      // The level's nodes with records: row start and degree prefix. The pairs
      // of a level are at most the CSR's records, so their number fits 31 bits
      // unless rows of an inconsistent CSR overlap. The sum of NT degrees is
      // known exactly all the same: its low 32 bits from the prefix sum, the
      // rest from the sum of the degrees' bits above 21 (below, each adds less
      // than 2^21, NT of them less than 2^31), which shares the second scan.
      constexpr int kHighShift = 21, kNodeBits = 11;
      static_assert(NT == 1 << 10 && NT < 1 << kNodeBits, "room for the node count below the degrees' high bits");
      int32_t carry = 0, nx = 0;
      for (int32_t c0 = 0; c0 < nlev; c0 += NT) {
        const int32_t i = c0 + t;
        int32_t d = 0, lo = 0;
        if (i < nlev) {
          const int32_t u = ent[lb + i];
          lo = a.row_ptr[u];
          const int32_t hi = a.row_ptr[u + 1];
          if (uint32_t(lo) <= uint32_t(hi) && uint32_t(hi) <= E) d = hi - lo;
          else flags |= RDF2V_STATUS_BAD_CSR;
        }
        int32_t tot, both;
        const int32_t ex = block_scan<NT>(d, scratch(), tot);
        const int32_t at = nx + (block_scan<NT>((d > 0 ? 1 : 0) + ((d >> kHighShift) << kNodeBits), scratch(), both) &
                                 ((1 << kNodeBits) - 1));
        const uint32_t high = uint32_t(both) >> kNodeBits;
        const int64_t records = (int64_t(high) << kHighShift) + (uint32_t(tot) - (high << kHighShift));
        if (carry + records > int64_t(E)) {  // uniform
          overlap = true;
          break;
        }
        if (d > 0) {
          x_node[at] = lb + i;
          x_lo[at] = lo;
          x_pre[at] = carry + ex;
        }
        carry += tot;
        nx += both & ((1 << kNodeBits) - 1);
      }
      if (overlap) break;
      const int32_t total = carry;
      int32_t added = 0;  // nodes of the next level so far (at the depth limit: up to max_walks or a batch more)
      int32_t more = 0;   // whether this thread reached one that was not counted
      __syncthreads();
      for (int32_t i0 = 0; i0 < nx && !overflow; i0 += kWideWindow) {
        // The next kWideWindow of them: their prefix, rows and child marks in LDS.
        const int32_t nw = min(kWideWindow, nx - i0);
        if (t < nw) {
          win_pre[t] = uint32_t(x_pre[i0 + t]);
          win_lo[t] = x_lo[i0 + t];
          win_child[t] = 0;
        } else if (t < kWideWindow) {
          win_pre[t] = 0xFFFFFFFFu;
        }
        if (t < kWave) win_pre[kWideWindow + t] = 0xFFFFFFFFu;
        const uint32_t q_end = uint32_t(i0 + nw < nx ? x_pre[i0 + nw] : total);
        __syncthreads();
        // The window node of pair q (uniform): the largest whose prefix is at
        // most q, from 64 samples and the 16 entries after the last that is.
        auto node_of = [&](uint32_t q) -> int32_t {
          constexpr int kStep = kWideWindow / kWave;
          const int32_t s = (__popcll(__ballot(win_pre[lane_id() * kStep] <= q)) - 1) * kStep;
          return s + __popcll(__ballot(lane_id() < kStep && win_pre[s + lane_id() % kStep] <= q)) - 1;
        };
        for (uint32_t c0 = win_pre[0]; c0 < q_end;) {
          const bool marks_only = last && added >= a.max_walks;  // uniform
          if (marks_only) {
            // Every walk of the depth limit is known: what is left to learn is
            // which nodes still reach something new. On one long row that
            // takes no order, so it streams through without a barrier.
            const int32_t n = node_of(c0);
            const uint32_t row_end = min(win_pre[n + 1], q_end);
            if (row_end - c0 >= uint32_t(kWideStreamRow)) {
              const uint32_t j0 = uint32_t(win_lo[n]) - win_pre[n];
              bool any = false;
              for (uint32_t q0 = c0 + uint32_t(t); q0 < row_end; q0 += kWideChunk) {
                int32_t x[R];
#pragma unroll
                for (int k = 0; k < R; ++k) {
                  const uint32_t q = q0 + uint32_t(k * NT);
                  x[k] = -1;
                  if (q < row_end && j0 + q < E) x[k] = edges[j0 + q].y;
                  else if (k > 0) x[k] = x[0];
                }
#pragma unroll
                for (int k = 0; k < R; ++k) {
                  if (uint32_t(x[k]) >= uint32_t(V)) flags |= RDF2V_STATUS_ID_OUT_OF_RANGE;
                  else if (!visited(x[k])) {
                    visit(x[k]);
                    any = true;
                  }
                }
              }
              if (any) {
                win_child[n] = 1;
                more = 1;
              }
              c0 = row_end;
              __syncthreads();
              continue;
            }
          }
          // Filter: wave w takes pairs c0 + w * 64 R + k * 64 + lane.
          int32_t node_k[R];
          int2 rec_k[R];
          uint32_t mask = 0;
          const uint32_t first = c0 + uint32_t(wave_index() * kWave * R);
#pragma unroll
          for (int k = 0; k < R; ++k) {
            node_k[k] = -1;
            rec_k[k] = make_int2(0, -1);
          }
          if (first < q_end) {  // uniform
            int32_t n0 = node_of(first);
            int32_t n[R];
#pragma unroll
            for (int k = 0; k < R; ++k) n[k] = n0;
            if (win_pre[n0 + 1] < first + kWave * R) {  // uniform: the wave's pairs cross a row's end
              // Per round, the rows that begin among its 64 pairs (at most 64,
              // each at a pair of its own) as a mask of those pairs.
#pragma unroll
              for (int k = 0; k < R; ++k) {
                const uint32_t at = win_pre[n0 + 1 + lane_id()] - (first + uint32_t(k * kWave));
                const uint32_t lo = wave_sum(at < 32u ? 1u << at : 0u);
                const uint32_t hi = wave_sum(at - 32u < 32u ? 1u << (at - 32u) : 0u);
                const uint64_t begins = (uint64_t(hi) << 32) | lo;
                n[k] = min(n0 + lanes_below(begins) + int32_t((begins >> lane_id()) & 1u), nw - 1);
                n0 = min(n0 + __popcll(begins), nw - 1);
              }
            }
#pragma unroll
            for (int k = 0; k < R; ++k) {
              const uint32_t q = first + uint32_t(k * kWave + lane_id());
              const uint32_t j_rec = uint32_t(win_lo[n[k]]) + (q - win_pre[n[k]]);
              if (q < q_end && j_rec < E) {  // below E in a consistent CSR
                node_k[k] = n[k];
                rec_k[k] = edges[j_rec];
              }
            }
          }
#pragma unroll
          for (int k = 0; k < R; ++k) {
            if (node_k[k] < 0) continue;
            if (uint32_t(rec_k[k].y) >= uint32_t(V)) flags |= RDF2V_STATUS_ID_OUT_OF_RANGE;
            else if (!visited(rec_k[k].y)) mask |= 1u << k;
          }
          int32_t rank[R], cands;
          rank_wide_chunk<NT, R>(mask, rank, cands, scratch());
          // Settle the candidates NT at a time, in pair order.
          for (int32_t base = 0; base < cands && !overflow; base += NT) {
            for (int i = t; i < kWideSlots; i += NT) table[i] = 0;
#pragma unroll
            for (int k = 0; k < R; ++k) {
              const int32_t at = rank[k] - base;
              if (((mask >> k) & 1u) && at >= 0 && at < NT) {
                c_ent[at] = rec_k[k].y;
                c_pred[at] = rec_k[k].x;
                c_node[at] = node_k[k];
              }
            }
            __syncthreads();
            const int32_t n_batch = min(cands - base, NT);
            int32_t slot = -1, x = 0;
            if (t < n_batch) {
              x = c_ent[t];
              // an earlier batch of this chunk may have reached it since
              if (base == 0 || !visited(x)) {
                slot = entity_slot<11>(x);
                static_assert(kWideSlots == 1 << 11, "entity_slot's table size");
                for (;;) {  // ends: the table has twice as many slots as candidates
                  const uint32_t cur = atomicCAS(&table[slot], 0u, uint32_t(t) + 1u);
                  if (cur == 0u) break;
                  if (c_ent[cur - 1] == x) {
                    atomicMin(&table[slot], uint32_t(t) + 1u);
                    break;
                  }
                  slot = (slot + 1) & (kWideSlots - 1);
                }
              }
            }
            __syncthreads();
            const bool win = slot >= 0 && table[slot] == uint32_t(t) + 1u;
            int32_t ex = 0, tot = 0, keep = 0;  // keep: nodes to store
            if (!marks_only) {
              ex = block_scan<NT>(win ? 1 : 0, scratch(), tot);
              keep = last ? min(tot, max(0, a.max_walks - added)) : tot;
            }
            if (keep > 0 && int64_t(le) + added + keep > p.node_cap) {  // uniform
              overflow = true;
            } else if (win) {
              visit(x);
              win_child[c_node[t]] = 1;
              if (marks_only) more = 1;
              if (ex < keep) {
                const int32_t pos = le + added + ex;
                ent[pos] = x;
                parent[pos] = x_node[i0 + c_node[t]];
                pred[pos] = c_pred[t];
                has_child[pos] = 0;
              }
            }
            added += tot;
            __syncthreads();
          }
          if (overflow) break;
          c0 += kWideChunk;
        }
        if (t < nw && win_child[t]) has_child[x_node[i0 + t]] = 1;
        __syncthreads();
      }
      if (overflow) break;
      if (last) {
        last_wins = added;
        if (added >= a.max_walks && __syncthreads_or(more)) last_wins = max(added, a.max_walks + 1);
      } else {
        lb = le;
        le += added;
        if (added > 0) {
          ++levels;
          if (t == 0) level_begin[levels] = le;
        }
        __syncthreads();
      }
    }
    if (overflow) {
      if (t == 0 && p.out_queue != nullptr) p.out_queue[atomicAdd(p.out_count, 1)] = int32_t(r);
      __syncthreads();
      continue;
    }
    if (overlap) {
      if (t == 0) a.counts[r] = 0;
      flags |= RDF2V_STATUS_BAD_CSR;
      __syncthreads();
      continue;
    }
    // Walks: the leaves among the stored levels in the order reached, then the
    // entities at the depth limit.
    int32_t leaves = 0;
    const int32_t kept_last = min(last_wins, a.max_walks);
    for (int32_t c0 = 0; c0 < le + kept_last && leaves <= a.max_walks; c0 += NT) {
      const int32_t i = c0 + t;
      const bool deep = i >= le;  // at the depth limit
      const int32_t leaf = i < le + kept_last ? int32_t(deep || has_child[i] == 0) : 0;
      int32_t tot;
      const int32_t ex = block_scan<NT>(leaf, scratch(), tot);
      const int32_t idx = leaves + ex;
      if (leaf && idx < a.max_walks) {
        int32_t h = a.depth;
        if (!deep) {
          h = 0;
          while (h + 1 < levels && level_begin[h + 1] <= i) ++h;
        }
        int32_t *row = a.tokens + (r * a.max_walks + idx) * width;
        int32_t node = i;
        for (int32_t step = h; step >= 1; --step) {
          row[2 * step] = ent[node];
          row[2 * step - 1] = V + pred[node];
          node = parent[node];
        }
        row[0] = root;
        for (int64_t j = 2 * int64_t(h) + 1; j < width; ++j) row[j] = -1;
        a.lens[r * a.max_walks + idx] = 2 * h + 1;
      }
      leaves += tot;
    }
    // `leaves` now counts every walk, or more than max_walks; entities at the
    // depth limit beyond those kept make the root over-full as well.
    if (t == 0) {
      a.counts[r] = min(leaves, a.max_walks);
      if (leaves > a.max_walks || last_wins > kept_last) flags |= RDF2V_STATUS_CAPACITY;
    }
    __syncthreads();
  }
  if (flags && a.status != nullptr) atomicOr(a.status, flags);
}

// The rows past counts[r] of a root: one contiguous range of tokens and one of
// lengths, filled with 16-byte stores between their ends, a wave's stores at
// whole 128-byte lines. Bound by HBM writes where they are many (100K roots of
// the 1M-triple uniform graph, depth 3, 14 % of 3.3 GB left unused: 93 us, against
// 478 us for filling everything beforehand; 26,230 roots with 97 % of 644 MB unused:
// 126 us, where a fill of everything takes 99, its waves following the address 4
// KB each; done like that here, the waves that find used rows cost 218 us in the
// first case).
// 2^lane_bits threads of a workgroup take a root, fewer where a root's rows are few
// (100K roots of 8 rows of 3 tokens: 73 -> 10 us within a call, from a workgroup
// each), and 2^slice_bits workgroups share one where there are fewer roots than fill
// the chip (one root of 1M rows of 9: 301 -> 18 us).
// kPast: the stores go past the caches. That is faster for what does not fit
// the Infinity Cache (459 MB: 93 us, 143 with plain stores) and slower for what
// does (163 MB: 36 us, 30 with plain ones; 99 MB: 24.6, 18.8; 36 MB: equal).
template <bool kPast>
__device__ __forceinline__ void fill_run(int32_t *p, int64_t count, int32_t value, int32_t t, int32_t lanes) {
  typedef int32_t v4i32 __attribute__((ext_vector_type(4)));
  const int32_t shift = int32_t((reinterpret_cast<uintptr_t>(p) & 127) >> 2);  // ints into a 128-byte line
  int32_t *line = p - shift;
  const int64_t end = shift + count, g0 = (shift + 3) >> 2, g1 = end >> 2;  // whole groups of four ints
  for (int64_t g = t; g < g1; g += lanes) {
    const v4i32 v = {value, value, value, value};
    if (g < g0) continue;
    if (kPast) __builtin_nontemporal_store(v, reinterpret_cast<v4i32 *>(line) + g);
    else reinterpret_cast<v4i32 *>(line)[g] = v;
  }
  // the ints before the first and behind the last of them
  if (t < 8) {
    const int64_t q = t < 4 ? 4 * g0 - 4 + t : 4 * max(g0, g1) + (t - 4);
    if (q >= shift && q < end) line[q] = value;
  }
}

constexpr int kFillThreads = 256;
constexpr int kFillLeastLaneBits = 3;   // 8 lanes for the three ints before and behind the 16-byte stores
constexpr int64_t kFillSliceInts = 4096;
constexpr int64_t kFillMostSliced = 65536;  // workgroups that slices add up to at most
static_assert(kFillSliceInts >= 8 * kFillThreads, "a sliced root has a workgroup to a slice");
constexpr int64_t kFillCachedInts = int64_t(56) << 20;  // 7/8 of the Infinity Cache's 256 MB

template <bool kPast>
__global__ __launch_bounds__(kFillThreads) void bfs_fill_unused_kernel(const int32_t *__restrict__ counts,
                                                                       int64_t num_roots, int32_t max_walks, int32_t width,
                                                                       int32_t lane_bits, int32_t slice_bits, int32_t slice_rows,
                                                                       int32_t *__restrict__ tokens,
                                                                       int32_t *__restrict__ lens) {
  const int32_t lanes = 1 << lane_bits, t = threadIdx.x & (lanes - 1);
  const uint32_t slice = blockIdx.x & ((1u << slice_bits) - 1);
  const int32_t first = int32_t(min(slice * uint32_t(slice_rows), uint32_t(max_walks)));
  const int32_t end = first + min(max_walks - first, slice_rows);
  const int32_t step = int32_t(gridDim.x >> slice_bits) * (kFillThreads >> lane_bits);
  const int32_t r0 = int32_t(blockIdx.x >> slice_bits) * (kFillThreads >> lane_bits) + int32_t(threadIdx.x >> lane_bits);
  for (int64_t r = r0; r < num_roots; r += step) {
    const int32_t lo = min(max(counts[r], first), end);
    const int64_t row = r * max_walks + lo;
    fill_run<kPast>(tokens + row * width, int64_t(end - lo) * width, -1, t, lanes);
    fill_run<kPast>(lens + row, end - lo, 0, t, lanes);
  }
}

}  // namespace

rdf2v_status launch_bfs_fill_unused(const int32_t *counts, int64_t num_roots, int32_t max_walks, int32_t width,
                                    int32_t *tokens_out, int32_t *len_out, hipStream_t stream) {
  const int64_t ints = int64_t(max_walks) * width;  // of one root
  int lane_bits = kFillLeastLaneBits;  // up to two 16-byte stores a lane
  while (1 << lane_bits < kFillThreads && ints > int64_t(8) << lane_bits) ++lane_bits;
  int slice_bits = 0;  // slices of about kFillSliceInts
  while (ints > kFillSliceInts << slice_bits && num_roots << slice_bits < kFillMostSliced / 2) ++slice_bits;
  const int32_t slice_rows = int32_t((int64_t(max_walks) + (int64_t(1) << slice_bits) - 1) >> slice_bits);
  const int64_t per_block = kFillThreads >> lane_bits;
  const int64_t blocks = std::min<int64_t>((num_roots + per_block - 1) / per_block, int64_t(1) << 20) << slice_bits;
  const bool cached = ints + max_walks <= kFillCachedInts / num_roots;
  auto kernel = cached ? bfs_fill_unused_kernel<false> : bfs_fill_unused_kernel<true>;
  kernel<<<dim3(unsigned(blocks)), dim3(kFillThreads), 0, stream>>>(counts, num_roots, max_walks, width, lane_bits,
                                                                   slice_bits, slice_rows, tokens_out, len_out);
  RDF2V_LAUNCH_CHECK();
  return RDF2V_OK;
}

template <class T>
void launch_tier(const BfsArgs &a, const int32_t *in_q, const int32_t *in_c, int32_t *taken, int32_t *out_q,
                 int32_t *out_c, int64_t grid, hipStream_t stream) {
  bfs_lds_kernel<T::kThreads, T::kRounds, T::kLog, T::kCap, T::kTreeCap, T::kWavesPerSimd>
      <<<dim3(unsigned(grid)), dim3(T::kThreads), 0, stream>>>(a, in_q, in_c, taken, out_q, out_c);
}

// The tier every root starts in: the smallest whose capacity is at least twice
// the expected tree size, 1 + d + ... + d^depth for the mean out-degree d
// (at most V). Only the speed depends on this choice: a root that outgrows a
// tier is rerun by the next.
int bfs_first_tier(int32_t num_entities, int64_t num_edges, int64_t num_roots, int32_t depth) {
  const double d = num_entities > 0 ? double(num_edges) / double(num_entities) : 0.0;
  double est = 1.0, level = 1.0;
  for (int32_t l = 0; l < depth && est < 1e9; ++l) {
    level *= d;
    est += level;
  }
  est = std::min(est, double(num_entities));
  int first = 2.0 * est <= TinyTier::kCap ? 0 : 2.0 * est <= SmallTier::kCap ? 1 : 2;
  // When a tier with more threads per root holds every root on the chip at
  // once, the extra threads shorten each root instead of waiting.
  int cus = 0, dev = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    cus = 0;
  if (first < 2 && num_roots <= int64_t(cus) * BigTier::kPerCu) first = 2;
  else if (first < 1 && num_roots <= int64_t(cus) * SmallTier::kPerCu) first = 1;
  return first;
}

int64_t bfs_workspace_units(int32_t num_entities, int64_t num_roots) {
  const int64_t per = int64_t(slice_bytes(num_entities));
  int64_t g = std::max<int64_t>(1, (int64_t(1) << 32) / std::max<int64_t>(per, 1));
  g = std::min<int64_t>(g, 2048);
  g = std::min<int64_t>(g, std::max<int64_t>(num_roots, 1));
  return g;
}

size_t bfs_walks_workspace_bytes(int32_t num_entities, int64_t num_roots) {
  return queue_bytes(num_roots) + size_t(bfs_workspace_units(num_entities, num_roots)) * slice_bytes(num_entities);
}

// The bitmap pass over queue 2 (an empty queue costs one load per workgroup).
// As many workgroups as the chip can hold, each with an equal slice of the
// workspace; slices smaller than V nodes send the roots that outgrow them to a
// second run with slices of V nodes (at least one fits: 36 bytes per entity
// against 25 and a bit).
rdf2v_status launch_wide(const BfsArgs &a, char *slices, size_t bytes, hipStream_t stream) {
  const int64_t V = a.num_entities;
  int lds = 0, cus = 0, dev = 0;
  RDF2V_HIP_TRY(hipGetDevice(&dev));
  RDF2V_HIP_TRY(hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
  RDF2V_HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  const size_t bitmap = wide_bitmap_bytes(V);
  const bool in_lds = bitmap + kWideStaticLds <= size_t(lds);
  const size_t head = in_lds ? 0 : bitmap;  // bytes of a slice before its nodes
  auto run = [&](WidePass p, int64_t groups) -> rdf2v_status {
    const dim3 grid{unsigned(groups)}, block{kWideThreads};
    if (in_lds) bfs_wide_kernel<true><<<grid, block, bitmap, stream>>>(a, p);
    else bfs_wide_kernel<false><<<grid, block, 0, stream>>>(a, p);
    RDF2V_LAUNCH_CHECK();
    return RDF2V_OK;
  };
  const int64_t per_cu = in_lds && 2 * (bitmap + kWideStaticLds) > size_t(lds) ? 1 : 2;
  int64_t groups = std::min<int64_t>(a.num_roots, std::max(1, cus) * per_cu);
  // at least 64K nodes (or V of them) per slice
  const int64_t least_nodes = std::min<int64_t>(V, 65536);
  const size_t least = head + wide_slice_bytes(least_nodes);
  groups = std::max<int64_t>(1, std::min<int64_t>(groups, int64_t(bytes / least)));
  WidePass p;
  p.in_queue = a.queue[2];
  p.in_count = a.queue_counts + 2;
  p.taken = a.queue_counts + kWideTaken;
  p.slices = slices;
  p.slice_bytes = bytes / size_t(groups) / 256 * 256;
  p.node_cap = int32_t(std::min<int64_t>(V, std::max(least_nodes, wide_slice_nodes(p.slice_bytes - head))));
  const bool all_fit = p.node_cap >= V;
  p.out_queue = all_fit ? nullptr : a.queue[0];
  p.out_count = all_fit ? nullptr : a.queue_counts + kWide2Length;
  const rdf2v_status st = run(p, groups);
  if (st != RDF2V_OK || all_fit) return st;
  p.in_queue = a.queue[0];
  p.in_count = a.queue_counts + kWide2Length;
  p.taken = a.queue_counts + kWide2Taken;
  p.slice_bytes = head + wide_slice_bytes(V);
  p.node_cap = int32_t(V);
  p.out_queue = p.out_count = nullptr;
  groups = std::max<int64_t>(1, std::min<int64_t>(groups, int64_t(bytes / p.slice_bytes)));
  return run(p, groups);
}

rdf2v_status launch_bfs_walks(const int32_t *row_ptr, const int32_t *edges, int64_t num_edges,
                              int32_t num_entities, int32_t num_predicates, const int32_t *roots,
                              int64_t num_roots, int32_t depth, int32_t max_walks, int32_t *tokens_out,
                              int32_t *len_out, int32_t *counts_out, void *workspace, int32_t *status_dev,
                              hipStream_t stream) {
  if (num_roots == 0) return RDF2V_OK;
  char *ws = static_cast<char *>(workspace);
  BfsArgs a;
  a.row_ptr = row_ptr;
  a.edges = edges;
  a.roots = roots;
  a.tokens = tokens_out;
  a.lens = len_out;
  a.counts = counts_out;
  a.status = status_dev;
  a.queue_counts = reinterpret_cast<int32_t *>(ws);
  for (int i = 0; i < 3; ++i) a.queue[i] = reinterpret_cast<int32_t *>(ws + 256 + i * align_up(size_t(num_roots) * 4, 256));
  a.num_roots = num_roots;
  a.num_edges = num_edges;
  a.num_entities = num_entities;
  a.num_predicates = num_predicates;
  a.depth = depth;
  a.max_walks = max_walks;
  bfs_queue_reset_kernel<<<1, kWave, 0, stream>>>(a.queue_counts);
  RDF2V_LAUNCH_CHECK();
  // The first tier takes every root, one per workgroup (the hardware hands
  // out roots as workgroups finish; at most 2^20 workgroups); a later tier
  // runs a grid over its input queue, whose length only the device knows, and
  // its workgroups past the end return at once.
  const int first = bfs_first_tier(num_entities, num_edges, num_roots, depth);
  for (int tier = first; tier < 3; ++tier) {
    const int32_t *in_q = tier == first ? nullptr : a.queue[tier - 1];
    const int32_t *in_c = tier == first ? nullptr : a.queue_counts + (tier - 1);
    const int64_t grid = std::min<int64_t>(num_roots, tier == first ? int64_t(1) << 20 : 2048);
    int32_t *taken = a.queue_counts + 3 + tier;
    if (tier == 0) launch_tier<TinyTier>(a, in_q, in_c, taken, a.queue[0], a.queue_counts + 0, grid, stream);
    else if (tier == 1) launch_tier<SmallTier>(a, in_q, in_c, taken, a.queue[1], a.queue_counts + 1, grid, stream);
    else launch_tier<BigTier>(a, in_q, in_c, taken, a.queue[2], a.queue_counts + 2, grid, stream);
    RDF2V_LAUNCH_CHECK();
  }
  return launch_wide(a, ws + queue_bytes(num_roots),
                     size_t(bfs_workspace_units(num_entities, num_roots)) * slice_bytes(num_entities), stream);
}

}  // namespace rdf2v
