// Skip-gram training pairs and CBOW training examples from walk rows on gfx950.
//
// gpuRDF2vec turns the walk corpus into center-context pairs for SkipGram
// (Sec. 3.2) after dropping the -1 padding (Sec. 3.1). For walk r with
// L = len[r] valid tokens t_0 .. t_{L-1}, every center i and every context j
// with 1 <= |i - j| <= window, 0 <= j < L, give the pair (t_i, t_j), ordered
// by walk, then i, then j.
//
// The number of pairs of a walk is a closed form of L and the window, so the
// output offsets are one exclusive scan and the emit kernels need no atomics: a
// block of them takes a few walks, learns its first output from the scan of the
// blocks' counts (int64: a corpus easily exceeds 2^31 pairs), and its walks'
// and centers' places follow in closed form. Pure integer streaming work, bound
// by HBM writes.
//
// CBOW (Sec. 3.2: the library trains Continuous Bag of Words next to
// Skip-Gram; it predicts a center token from the tokens around it) takes one
// example per valid token: the center t_i and its contexts, the t_j with
// 1 <= |i - j| <= window in ascending j, padded with -1 to 2 * window entries.
// Examples are ordered by walk, then i; a walk of L tokens gives L of them, so
// the offsets are a scan of the lengths and the same kernels serve both.

#include <algorithm>

#include "common.hpp"
#include "grid.hpp"
#include "launch.hpp"

namespace rdf2v {
namespace {

typedef int32_t v4i32 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kCountThreads = 1024;  // of a workgroup that counts emit blocks

// All arithmetic inside a block is 32-bit: a walk has at most 129 tokens, a
// block at most 32,768 items, and the window is clamped to the row (a wider
// one reaches no further).
__device__ __forceinline__ int32_t clamp_window(int32_t window, int32_t width) { return min(window, width); }

// Pairs of a walk with L valid tokens: 2 * sum_{d=1}^{m} (L - d), m = min(window, L - 1).
__device__ __forceinline__ int32_t walk_pairs(int32_t L, int32_t window) {
  const int32_t m = min(window, L - 1);
  return m <= 0 ? 0 : m * (2 * L - m - 1);
}

// sum_{k=0}^{n-1} min(k, window)
__device__ __forceinline__ int32_t capped_prefix(int32_t n, int32_t window) {
  if (n <= 0) return 0;
  if (n <= window + 1) return n * (n - 1) / 2;
  return window * (window + 1) / 2 + (n - 1 - window) * window;
}

// Training items of one walk of L valid tokens: pairs, or CBOW examples.
template <bool kCbow>
__device__ __forceinline__ int32_t walk_items(int32_t L, int32_t window) {
  return kCbow ? L : walk_pairs(L, window);
}

// A walk's length, clamped to the row; out-of-range lengths raise a flag.
__device__ __forceinline__ int32_t clamped(int32_t L, int32_t width, int &bad) {
  if (L < 0 || L > width) {
    bad = 1;
    return L < 0 ? 0 : width;
  }
  return L;
}

// Where the emit blocks' outputs begin: the items of `walks` consecutive walks
// (one emit block) per kLanes threads, their exclusive prefix inside the workgroup
// to firsts, the workgroup's total to partials. A lone workgroup also writes what
// partials_scan_kernel would.
template <bool kCbow, int kLanes>
__global__ __launch_bounds__(kCountThreads) void item_count_kernel(const int32_t *__restrict__ len, int64_t n,
                                                                   int32_t width, int32_t window, int32_t walks,
                                                                   int64_t emit_blocks, int32_t *__restrict__ firsts,
                                                                   int64_t *__restrict__ partials, int64_t *total_out,
                                                                   int32_t *status) {
  __shared__ int32_t scratch[kCountThreads / kWave];
  const int64_t b = int64_t(blockIdx.x) * (kCountThreads / kLanes) + threadIdx.x / kLanes;
  const int32_t lane = threadIdx.x % kLanes;
  const int32_t w = clamp_window(window, width);
  constexpr int32_t kAhead = 8;  // lengths of a thread in flight together
  int32_t s = 0;
  int bad = 0;
  if (b < emit_blocks) {
    const int64_t r0 = b * walks;
    const int32_t rows = int32_t(min(int64_t(walks), n - r0));
    for (int32_t i0 = lane; i0 < rows; i0 += kAhead * kLanes) {
      int32_t L[kAhead];
#pragma unroll
      for (int32_t k = 0; k < kAhead; ++k) L[k] = i0 + k * kLanes < rows ? len[r0 + i0 + k * kLanes] : 0;
#pragma unroll
      for (int32_t k = 0; k < kAhead; ++k) s += walk_items<kCbow>(clamped(L[k], width, bad), w);
    }
  }
#pragma unroll
  for (int32_t off = 1; off < kLanes; off <<= 1) s += __shfl_xor(s, off, kWave);
  int32_t total;
  const int32_t ex = block_exclusive_scan<kCountThreads>(lane == 0 ? s : 0, scratch, total);
  if (b < emit_blocks && lane == 0) firsts[b] = ex;
  if (threadIdx.x == 0) {
    partials[blockIdx.x] = gridDim.x == 1 ? 0 : total;
    if (gridDim.x == 1) *total_out = total;
  }
  if (bad && status != nullptr) atomicOr(status, RDF2V_STATUS_BAD_LENGTH);
}

// One block: exclusive scan of the workgroup totals in place; the sum goes to *total_out.
__global__ __launch_bounds__(kCountThreads) void partials_scan_kernel(int64_t *partials, int64_t nb,
                                                                      int64_t *total_out) {
  __shared__ int64_t scratch[kCountThreads / kWave];
  int64_t carry = 0;
  for (int64_t base = 0; base < nb; base += kCountThreads) {
    const int64_t idx = base + threadIdx.x;
    const int64_t x = idx < nb ? partials[idx] : 0;
    int64_t tot;
    const int64_t ex = block_exclusive_scan<kCountThreads, int64_t>(x, scratch, tot);
    if (idx < nb) partials[idx] = carry + ex;
    carry += tot;
  }
  if (threadIdx.x == 0) *total_out = carry;
}

// What an emit block works on, shared by the emit kernels: its walk rows and,
// per walk, the valid length and where its items begin inside the block.
template <int kBlock>
struct BlockWalks {
  int32_t rows[kBlock];
  int32_t lens[kBlock];
  int32_t firsts[kBlock];
  int32_t scan[kBlock / kWave];
};

struct EmitArgs {
  const int32_t *tokens;
  const int32_t *len;
  int64_t n;
  int32_t width, window;
  int32_t walks;              // per emit block: kBlock / width
  uint32_t width_inverse;     // ceil(2^32 / width); 0 for width 1
  const int32_t *firsts;
  const int64_t *partials;    // per 2^group_bits emit blocks
  int32_t group_bits;
  int64_t capacity;
  int32_t *status;
};

// t / width for t below the block size.
__device__ __forceinline__ int32_t walk_of(const EmitArgs &a, int32_t t) {
  return a.width == 1 ? t : int32_t(__umulhi(uint32_t(t), a.width_inverse));
}

// Fills s for block blockIdx.x (every global read of the block is issued
// before the first barrier), ends with a barrier, and returns the number of
// the block's items; first: the first of them in the output.
template <bool kCbow, int kBlock>
__device__ __forceinline__ int32_t load_walks(const EmitArgs &a, BlockWalks<kBlock> &s, int64_t &first) {
  const int32_t t = threadIdx.x;
  const int64_t r0 = int64_t(blockIdx.x) * a.walks;
  const int32_t walks = int32_t(min(int64_t(a.walks), a.n - r0));
  first = a.partials[blockIdx.x >> a.group_bits] + a.firsts[blockIdx.x];
  int bad = 0;  // reported by the count
  const int32_t token = t < walks * a.width ? a.tokens[r0 * a.width + t] : 0;
  const int32_t L = t < walks ? clamped(a.len[r0 + t], a.width, bad) : 0;
  const int32_t items = walk_items<kCbow>(L, clamp_window(a.window, a.width));
  s.rows[t] = token;
  s.lens[t] = L;
  int32_t total;
  if (kBlock == kWave || a.walks <= kWave) {  // uniform: the first wave holds every walk
    const int32_t v = wave_inclusive_sum(items);
    if (t < kWave) s.firsts[t] = v - items;
    if (t == kWave - 1) s.scan[0] = v;
    __syncthreads();
    total = s.scan[0];
  } else {
    s.firsts[t] = block_exclusive_scan<kBlock>(items, s.scan, total);
    __syncthreads();
  }
  return total;
}

// Streams ints [shift, shift + total) of an LDS stage to dst and on, where
// shift is dst's offset from 128-byte alignment in ints: the stage has the same
// offset, so what lies between the ends are 16-byte loads from LDS and 16-byte
// non-temporal stores, and every wave's store covers whole 128-byte lines
// (8M walks of 17 tokens, window 5: pairs 2.00 -> 1.69 ms, 4M: CBOW 0.63 -> 0.58
// ms against alignment to 16 bytes; plain stores 1.62 and 0.74).
constexpr int kLineInts = 32;
template <int kBlock>
__device__ __forceinline__ void stream_out(const int32_t *stage, int32_t shift, int32_t *dst, int32_t total) {
  const int32_t t = threadIdx.x;
  int32_t *base = dst - shift;
  const int32_t end = shift + total;
  const int32_t g0 = (shift + 3) >> 2, g1 = end >> 2;  // whole groups of four ints
  const v4i32 *src4 = reinterpret_cast<const v4i32 *>(stage);
  v4i32 *dst4 = reinterpret_cast<v4i32 *>(base);
  for (int32_t g = t; g < g1; g += kBlock)
    if (g >= g0) __builtin_nontemporal_store(src4[g], dst4 + g);
  // the ints before the first and behind the last of them
  if (t < 8) {
    const int32_t q = t < 4 ? 4 * g0 - 4 + t : 4 * max(g0, g1) + (t - 4);
    if (q >= shift && q < end) __builtin_nontemporal_store(stage[q], base + q);
  }
}
__device__ __forceinline__ int32_t int_shift(const void *p) {
  return int32_t((reinterpret_cast<uintptr_t>(p) & (4 * kLineInts - 1)) >> 2);
}

// Pairs: one thread per (walk, center). With kStage the threads place their
// pairs in an LDS stage sized at launch to the block's most pairs (dynamic
// LDS), and the block streams its contiguous range out; otherwise each thread
// writes its pairs directly, with plain stores (57K rows of 129 tokens, window
// 20: 1.1 ms, 12.1 with stores past the caches, 10.1-11.1 before rows were staged).
template <bool kStage, int kBlock>
__global__ __launch_bounds__(kBlock) void pair_emit_kernel(const EmitArgs a, int2 *__restrict__ pairs) {
  extern __shared__ __align__(16) int2 stage[];  // kStage: the block's pairs, from the offset of its range on
  __shared__ BlockWalks<kBlock> s;
  const int32_t t = threadIdx.x;
  const int32_t w = clamp_window(a.window, a.width);
  int64_t block_first;
  const int32_t total = load_walks<false>(a, s, block_first);
  const int64_t room = max(int64_t(0), a.capacity - block_first);
  int2 *dst = pairs + block_first;
  const int32_t shift = kStage ? int_shift(dst) : 0;
  const int32_t k_walk = walk_of(a, t), i = t - k_walk * a.width;
  // threads past the last walk (s.lens is 0 there) and past a walk's end have no center
  if (k_walk < a.walks && i < s.lens[k_walk]) {
    const int32_t L = s.lens[k_walk];
    const int32_t *row = s.rows + k_walk * a.width;
    const int32_t center = row[i];
    int32_t k = s.firsts[k_walk] + capped_prefix(i, w) + capped_prefix(L, w) - capped_prefix(L - i, w);
    const int32_t j0 = max(0, i - w), j1 = min(L - 1, i + w);
    int2 *out = stage + (shift >> 1);
    for (int32_t j = j0; j <= j1; ++j) {
      if (j == i) continue;
      const int2 pr = make_int2(center, row[j]);
      if (kStage) {
        out[k] = pr;
      } else if (k < room) {
        dst[k] = pr;  // through the caches, where pairs of eight bytes meet in whole lines
      }
      ++k;
    }
  }
  if (kStage) {
    __syncthreads();
    stream_out<kBlock>(reinterpret_cast<const int32_t *>(stage), shift, reinterpret_cast<int32_t *>(dst),
                       2 * int32_t(min(int64_t(total), room)));
  }
  if (total > room && t == 0 && a.status != nullptr) atomicOr(a.status, RDF2V_STATUS_CAPACITY);
}

// CBOW, staged: one thread per (walk, position), whose examples form one
// contiguous output range. The block places its centers and context rows in
// LDS stages (at most kBlock examples, 2 * window ints per context row) and
// streams each out.
template <int kBlock>
__global__ __launch_bounds__(kBlock) void cbow_emit_kernel(const EmitArgs a, int32_t *__restrict__ centers,
                                                            int32_t *__restrict__ contexts) {
  extern __shared__ __align__(16) int32_t ctx_stage[];        // the block's context rows, from their range's offset on
  __shared__ __align__(16) int32_t ctr_stage[kBlock + kLineInts];     // the block's centers, likewise
  __shared__ BlockWalks<kBlock> s;
  const int32_t t = threadIdx.x;
  int64_t block_first;
  const int32_t total = load_walks<true>(a, s, block_first);
  const int32_t w = a.window, cw = 2 * w;
  int32_t *ctr = centers + block_first;
  int32_t *ctx = contexts + block_first * cw;
  const int32_t ctr_shift = int_shift(ctr), ctx_shift = int_shift(ctx);
  const int32_t k_walk = walk_of(a, t), i = t - k_walk * a.width;
  if (k_walk < a.walks && i < s.lens[k_walk]) {
    const int32_t L = s.lens[k_walk];
    const int32_t *row = s.rows + k_walk * a.width;
    const int32_t e = s.firsts[k_walk] + i;
    ctr_stage[ctr_shift + e] = row[i];
    int32_t *out = ctx_stage + ctx_shift + e * cw;
    const int32_t j0 = max(0, i - w), nleft = i - j0, nctx = min(L - 1, i + w) - j0;
    for (int32_t m = 0; m < cw; ++m) out[m] = m < nctx ? row[j0 + m + (m < nleft ? 0 : 1)] : -1;
  }
  __syncthreads();
  // the examples that fit
  const int64_t room = max(int64_t(0), a.capacity - block_first);
  const int32_t lim = int32_t(min(int64_t(total), room));
  stream_out<kBlock>(ctr_stage, ctr_shift, ctr, lim);
  stream_out<kBlock>(ctx_stage, ctx_shift, ctx, lim * cw);
  if (total > room && t == 0 && a.status != nullptr) atomicOr(a.status, RDF2V_STATUS_CAPACITY);
}

// CBOW, written in output order. The block stages only its walk rows, their
// lengths and places, and the walk of each example; then every thread produces
// context entries directly in output order, four per 16-byte non-temporal
// store: entry m of example e is the m-th context of that example's position
// (the tokens j0 .. j1 of its window, skipping the position itself), or -1
// past the last one. No context row is ever staged, so the block's LDS does
// not grow with the window.
template <int kBlock>
__global__ __launch_bounds__(kBlock) void cbow_direct_kernel(const EmitArgs a, int32_t *__restrict__ centers,
                                                              int32_t *__restrict__ contexts) {
  __shared__ BlockWalks<kBlock> s;
  __shared__ int32_t ex_walk[kBlock];  // per example of the block: its walk
  const int32_t t = threadIdx.x;
  const int32_t width = a.width;
  int64_t block_first;
  const int32_t cnt = load_walks<true>(a, s, block_first);
  {
    const int32_t k_walk = walk_of(a, t), i = t - k_walk * width;
    if (k_walk < a.walks && i < s.lens[k_walk]) ex_walk[s.firsts[k_walk] + i] = k_walk;
  }
  __syncthreads();
  const int32_t *rows = s.rows, *walk_first = s.firsts, *walk_len = s.lens;
  const int64_t room = max(int64_t(0), a.capacity - block_first);
  const int32_t lim = int32_t(min(int64_t(cnt), room));  // those that fit
  const int32_t w = a.window, cw = 2 * w;
  // Centers: example e of the block is position e - walk_first of its walk.
  for (int32_t e = t; e < lim; e += kBlock) {
    const int32_t k = ex_walk[e];
    __builtin_nontemporal_store(rows[k * width + (e - walk_first[k])], centers + block_first + e);
  }
  // Context entry q = e * cw + m of the block; `next` steps to entry q + 1.
  struct Cursor {
    int32_t e, m, base, nleft, nctx;  // example, entry; the example's window start, contexts before / in all
  };
  auto at = [&](int32_t e, int32_t m) {
    Cursor c;
    c.e = e;
    c.m = m;
    const int32_t k = ex_walk[e];
    const int32_t pos = e - walk_first[k];
    const int32_t j0 = max(0, pos - w), j1 = min(walk_len[k] - 1, pos + w);
    c.base = k * width + j0;
    c.nleft = pos - j0;
    c.nctx = j1 - j0;
    return c;
  };
  auto value = [&](const Cursor &c) {
    return c.m < c.nleft ? rows[c.base + c.m] : (c.m < c.nctx ? rows[c.base + c.m + 1] : -1);
  };
  auto next = [&](Cursor &c) {
    if (++c.m == cw && c.e + 1 < lim) c = at(c.e + 1, 0);
  };
  const int32_t total = lim * cw;  // entries that fit (<= kBlock * 2 * RDF2V_MAX_DEPTH * 2)
  int32_t *dst = contexts + block_first * int64_t(cw);
  const int32_t head = min(total, int32_t(((16 - (reinterpret_cast<uintptr_t>(dst) & 15)) & 15) / 4));
  if (t < head) {
    const Cursor c = at(t / cw, t % cw);
    __builtin_nontemporal_store(value(c), dst + t);
  }
  const int32_t body = (total - head) >> 2;
  v4i32 *dst4 = reinterpret_cast<v4i32 *>(dst + head);
  for (int32_t q4 = t; q4 < body; q4 += kBlock) {
    const int32_t q = head + 4 * q4;
    Cursor c = at(q / cw, q % cw);
    v4i32 v;
    v.x = value(c);
    next(c);
    v.y = value(c);
    next(c);
    v.z = value(c);
    next(c);
    v.w = value(c);
    __builtin_nontemporal_store(v, dst4 + q4);
  }
  for (int32_t q = head + 4 * body + t; q < total; q += kBlock) {
    const Cursor c = at(q / cw, q % cw);
    __builtin_nontemporal_store(value(c), dst + q);
  }
  if (cnt > room && t == 0 && a.status != nullptr) atomicOr(a.status, RDF2V_STATUS_CAPACITY);
}

constexpr size_t kMaxStageBytes = 32 << 10, kBestStageBytes = 14 << 10;

// Most pairs one walk of this width can give.
inline int64_t max_walk_pairs(int64_t width, int64_t window) {
  const int64_t m = std::min(window, width - 1);
  return m <= 0 ? 0 : 2 * (m * width - m * (m + 1) / 2);
}

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

}  // namespace

// The size callers hold workspaces of: 8 bytes per walk and per 4,096 walks.
// What is kept in it are 4 bytes per emit block (one walk at least) and, behind
// them, 8 per kCountThreads of those.
size_t skipgram_workspace_bytes(int64_t num_walks) {
  const int64_t nb = ceil_div(num_walks, 4096);
  return align_up(size_t(num_walks) * 8, 256) + align_up(size_t(nb + 1) * 8, 256);
}

namespace {

// Counts the items of num_walks walks, `walks` of them per emit block, and
// fills the emit kernels' arguments.
template <bool kCbow>
rdf2v_status count_items(const int32_t *tokens, const int32_t *len, int64_t num_walks, int32_t width, int32_t window,
                         int32_t walks, int64_t capacity, int64_t *count_out, void *workspace, int32_t *status_dev,
                         hipStream_t stream, EmitArgs &a, int64_t &emit_blocks) {
  emit_blocks = ceil_div(num_walks, walks);
  if (emit_blocks >= (int64_t(1) << 31)) return RDF2V_ERR_TOO_LARGE;
  // One thread counts an emit block's walks, eight do where there are more than
  // 64 of them (rows of up to three tokens), which leave few emit blocks: 6M rows
  // of 3 tokens, window 2, 172 -> 114 us a call.
  const int32_t lanes = walks > kWave ? 8 : 1, group = kCountThreads / lanes;
  const int64_t nb = ceil_div(emit_blocks, group);
  int32_t *firsts = static_cast<int32_t *>(workspace);
  int64_t *partials = reinterpret_cast<int64_t *>(firsts + (emit_blocks + 1) / 2 * 2);
  a.tokens = tokens;
  a.len = len;
  a.n = num_walks;
  a.width = width;
  a.window = window;
  a.walks = walks;
  a.width_inverse = uint32_t(((uint64_t(1) << 32) + uint64_t(width) - 1) / uint64_t(width));
  a.firsts = firsts;
  a.partials = partials;
  a.group_bits = lanes == 1 ? 10 : 7;
  a.capacity = capacity;
  a.status = status_dev;
  if (nb > 0) {
    auto kernel = lanes == 1 ? item_count_kernel<kCbow, 1> : item_count_kernel<kCbow, 8>;
    kernel<<<dim3(unsigned(nb)), dim3(kCountThreads), 0, stream>>>(len, num_walks, width, window, walks, emit_blocks,
                                                                  firsts, partials, count_out, status_dev);
    RDF2V_LAUNCH_CHECK();
  }
  if (nb != 1) {
    partials_scan_kernel<<<dim3(1), dim3(kCountThreads), 0, stream>>>(partials, nb, count_out);
    RDF2V_LAUNCH_CHECK();
  }
  return RDF2V_OK;
}

// Runs emit(part, grid) over the emit blocks (of `threads` threads) in as few
// launches as HIP takes: a part's arguments begin at its first block.
template <class Emit>
rdf2v_status launch_emit(const EmitArgs &a, int64_t blocks, int threads, Emit emit) {
  return for_each_launch(blocks, threads, kCountThreads, [&](int64_t first, int64_t count) -> rdf2v_status {
    EmitArgs part = a;
    const int64_t r0 = first * a.walks;
    part.tokens += r0 * a.width;
    part.len += r0;
    part.n -= r0;
    part.firsts += first;
    part.partials += first >> a.group_bits;
    emit(part, dim3(unsigned(count)));
    RDF2V_LAUNCH_CHECK();
    return RDF2V_OK;
  });
}

}  // namespace

rdf2v_status launch_skipgram_pairs(const int32_t *tokens, const int32_t *len, int64_t num_walks,
                                   int32_t width, int32_t window, int32_t *pairs_out, int64_t capacity,
                                   int64_t *count_out, void *workspace, int32_t *status_dev,
                                   hipStream_t stream) {
  // The largest block whose pairs fit a stage of kBestStageBytes, else the
  // smallest that fits one of kMaxStageBytes: several small blocks per CU keep
  // the write stream going while others load rows and place pairs, down to
  // about 8 KB of output each (8M walks of 17 tokens, window 5: 1.55 ms with
  // 128 threads and 7.8 KB, 1.69 with 256 and 16.8, 1.68 with 64 and 3.4). Limits
  // of 7, 8, 10, 12 and 14 KB, over widths 1 to 129 and windows 1 to 64, differ by
  // no more than their runs do.
  const int64_t per_walk = max_walk_pairs(width, window);
  auto stage_bytes = [&](int block) { return size_t(per_walk * (block / width)) * sizeof(int2) + 4 * kLineInts; };
  int block = 0;  // 0: no stage
  for (int b : {64, 128, 256})
    if (width <= b && stage_bytes(b) <= (block == 0 ? kMaxStageBytes : kBestStageBytes)) block = b;
  EmitArgs a;
  int64_t blocks;
  const rdf2v_status st = count_items<false>(tokens, len, num_walks, width, window, (block ? block : kThreads) / width,
                                             capacity, count_out, workspace, status_dev, stream, a, blocks);
  if (st != RDF2V_OK || capacity == 0 || blocks == 0) return st;
  int2 *out = reinterpret_cast<int2 *>(pairs_out);
  return launch_emit(a, blocks, block ? block : kThreads, [&](const EmitArgs &p, dim3 grid) {
    if (block == 256) pair_emit_kernel<true, 256><<<grid, dim3(256), stage_bytes(256), stream>>>(p, out);
    else if (block == 128) pair_emit_kernel<true, 128><<<grid, dim3(128), stage_bytes(128), stream>>>(p, out);
    else if (block == 64) pair_emit_kernel<true, 64><<<grid, dim3(64), stage_bytes(64), stream>>>(p, out);
    else pair_emit_kernel<false, kThreads><<<grid, dim3(kThreads), 0, stream>>>(p, out);
  });
}

rdf2v_status launch_cbow_examples(const int32_t *tokens, const int32_t *len, int64_t num_walks, int32_t width,
                                  int32_t window, int32_t *centers_out, int32_t *contexts_out, int64_t capacity,
                                  int64_t *count_out, void *workspace, int32_t *status_dev, hipStream_t stream) {
  // The staged kernel holds a block's context rows in LDS, at most B rows of
  // 2 * window ints for B threads: 256 threads up to 14 KB, 128 up to 32 KB. The
  // output-order kernel needs no stage. us, staged / output order, for as many
  // rows of 17 tokens (9 tokens) as give about 1.2 GB, 6M at most:
  //   window 1: 481 / 533 (231 / 258)   2: 282 / 289 (256 / 264)   3: 239 / 273 (241 / 282)
  //          4: 248 / 228 (261 / 241)   5: 266 / 282 (273 / 289)   6: 255 / 279 (263 / 289)
  //          7: 281 / 294 (263 / 304)   8: 273 / 250 (274 / 259)  10: 259 / 283 (260 / 289)
  //         12: 257 / 273 (259 / 280)  16: 487 / 241 (492 / 248)  20: 247 / 280
  //         24: 296 / 246              32: 533 / 241
  // Threads place their context rows side by side, 2 * window banks apart, so
  // windows of a multiple of 8 queue at four banks or fewer and take the output
  // order, like window 4 and those whose stage does not fit.
  const bool staged = window % 8 != 0 && window != 4;
  const size_t row_bytes = size_t(2) * size_t(window) * sizeof(int32_t);
  auto stage_bytes = [&](int block) { return size_t(block / width * width) * row_bytes + 4 * kLineInts; };
  int block = 0;  // 0: output order
  for (int b : {128, 256})
    if (staged && width <= b && stage_bytes(b) <= (block == 0 ? kMaxStageBytes : kBestStageBytes)) block = b;
  EmitArgs a;
  int64_t blocks;
  const rdf2v_status st = count_items<true>(tokens, len, num_walks, width, window, (block ? block : kThreads) / width,
                                            capacity, count_out, workspace, status_dev, stream, a, blocks);
  if (st != RDF2V_OK || capacity == 0 || blocks == 0) return st;
  return launch_emit(a, blocks, block ? block : kThreads, [&](const EmitArgs &p, dim3 grid) {
    if (block == 256)
      cbow_emit_kernel<256><<<grid, dim3(256), stage_bytes(256), stream>>>(p, centers_out, contexts_out);
    else if (block == 128)
      cbow_emit_kernel<128><<<grid, dim3(128), stage_bytes(128), stream>>>(p, centers_out, contexts_out);
    else
      cbow_direct_kernel<kThreads><<<grid, dim3(kThreads), 0, stream>>>(p, centers_out, contexts_out);
  });
}

}  // namespace rdf2v
