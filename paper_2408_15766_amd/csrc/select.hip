// Selection kernels of the speculative-decoding cycle: vocabulary reductions (argmax,
// softmax statistics, top-k log-probabilities), the draft tree's candidate pool (expansion,
// frontier choice, rerank), acceptance (greedy walk, multi-round rejection sampling with a
// counter-based RNG) and the KV-cache compaction that commits the accepted path.
//
// Ordering rule everywhere: larger value first, equal values by lower index, so results are
// unique and independent of how the work is split over lanes.
#include <limits.h>

#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace spec {

constexpr int kSelThreads = 256;

// ---- counter-based RNG: splitmix64 finaliser chained over (seed, cycle, node, draw) --------
__device__ __forceinline__ uint64_t mix64(uint64_t x) {
  x ^= x >> 30; x *= 0xBF58476D1CE4E5B9ull;
  x ^= x >> 27; x *= 0x94D049BB133111EBull;
  x ^= x >> 31;
  return x;
}
__device__ __forceinline__ uint64_t rng_stream(uint64_t seed, uint32_t cycle, uint32_t node) {
  uint64_t s = mix64(seed + 0x9E3779B97F4A7C15ull);
  s = mix64(s + cycle);
  return mix64(s + node);
}
// 23 random bits centred in their cell: never 0 or 1, exact in fp32.
__device__ __forceinline__ float rng_uniform(uint64_t stream, uint64_t draw) {
  return ((float)(mix64(stream + draw) >> 41) + 0.5f) * 1.1920928955078125e-07f;
}
__device__ __forceinline__ float rng_gumbel(uint64_t stream, int v) {
  return -logf(-logf(rng_uniform(stream, (1ull << 32) + (uint64_t)v)));
}

// ---- per-row argmax ------------------------------------------------------------------------
// Stage 1: one workgroup per (slice of kTopkSlice entries, row) leaves the slice's best (value, index)
// in part_val / part_idx [rows][n_slices].  The consumer (greedy acceptance, or the finishing kernel)
// merges a row's slices with the same ordering rule, so the result is the row's first maximum.
__global__ __launch_bounds__(kSelThreads) void argmax_slice_kernel(const float *logits, int vocab, int n_slices,
                                                                   float *part_val, int *part_idx) {
  constexpr int PER = kTopkSlice / kSelThreads;   // 16
  __shared__ float shv[16];
  __shared__ int shi[16];
  const int slice = blockIdx.x, rowi = blockIdx.y, t = threadIdx.x;
  const int c0 = slice * kTopkSlice;
  const float *row = logits + (size_t)rowi * vocab;
  float v[PER];
#pragma unroll
  for (int e = 0; e < PER; e++) {
    const int c = c0 + t + e * kSelThreads;
    v[e] = c < vocab ? row[c] : -INFINITY;
  }
  ValIdx b{-INFINITY, INT_MAX};
#pragma unroll
  for (int e = 0; e < PER; e++) {
    const int c = c0 + t + e * kSelThreads;
    if (c < vocab && (v[e] > b.v || b.i == INT_MAX)) { b.v = v[e]; b.i = c; }   // ascending c: strict > keeps the lower index
  }
  b = block_best(b, shv, shi);
  if (t == 0) { part_val[(size_t)rowi * n_slices + slice] = b.v; part_idx[(size_t)rowi * n_slices + slice] = b.i; }
}
// One wavefront: best of a row's slice results.
__device__ __forceinline__ int merge_argmax(const float *part_val, const int *part_idx, int n_slices, int row, int lane) {
  ValIdx b{-INFINITY, INT_MAX};
  for (int sl = lane; sl < n_slices; sl += 64) {
    const float x = part_val[(size_t)row * n_slices + sl];
    const int c = part_idx[(size_t)row * n_slices + sl];
    if (better(x, c, b.v, b.i)) { b.v = x; b.i = c; }
  }
  return wave_best(b).i;
}
__global__ __launch_bounds__(64) void argmax_finish_kernel(const float *part_val, const int *part_idx, int n_slices, int *out) {
  const int best = merge_argmax(part_val, part_idx, n_slices, blockIdx.x, threadIdx.x);
  if (threadIdx.x == 0) out[blockIdx.x] = best;
}
int argmax_slices(int vocab) { return (vocab + kTopkSlice - 1) / kTopkSlice; }
hipError_t launch_rows_argmax(const float *logits, int rows, int vocab, float *part_val, int *part_idx, int *out,
                              hipStream_t st) {
  if (rows < 1 || vocab < 1) return hipErrorInvalidValue;
  const int n_slices = argmax_slices(vocab);
  hipLaunchKernelGGL(argmax_slice_kernel, dim3(n_slices, rows), dim3(kSelThreads), 0, st, logits, vocab, n_slices, part_val,
                     part_idx);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || out == nullptr) return e;
  hipLaunchKernelGGL(argmax_finish_kernel, dim3(rows), dim3(64), 0, st, part_val, part_idx, n_slices, out);
  return hipGetLastError();
}

// ---- per-row softmax statistics at temperature T, x = logit / T ----------------------------
// One workgroup per (slice of kTopkSlice entries, row): part[row][slice] = {max x, sum exp(x - max x)} over the
// slice.  merge_softmax_stats (one wavefront) turns a row's slices into {max x, sum exp(x - max x)} of the row.
__global__ __launch_bounds__(kSelThreads) void softmax_slice_kernel(const float *logits, int vocab, float temp, int n_slices,
                                                                    float2 *part) {
  constexpr int PER = kTopkSlice / kSelThreads;   // 16
  __shared__ float sh[16];
  const int slice = blockIdx.x, rowi = blockIdx.y, t = threadIdx.x;
  const int c0 = slice * kTopkSlice;
  const float *row = logits + (size_t)rowi * vocab;
  float v[PER];
#pragma unroll
  for (int e = 0; e < PER; e++) {
    const int c = c0 + t + e * kSelThreads;
    v[e] = c < vocab ? row[c] / temp : -INFINITY;
  }
  float m = v[0];
#pragma unroll
  for (int e = 1; e < PER; e++) m = fmaxf(m, v[e]);
  m = block_max(m, sh);
  float s = 0.f;
#pragma unroll
  for (int e = 0; e < PER; e++) s += expf(v[e] - m);        // exp(-inf) = 0 for padding
  s = block_sum(s, sh);
  if (t == 0) part[(size_t)rowi * n_slices + slice] = make_float2(m, s);
}
__device__ __forceinline__ float2 merge_softmax_stats(const float2 *part, int n_slices, int row, int lane) {
  const float2 *stat = part + (size_t)row * n_slices;
  float m = -INFINITY;
  for (int sl = lane; sl < n_slices; sl += 64) m = fmaxf(m, stat[sl].x);
  m = wave_max(m);
  float tot = 0.f;
  for (int s0 = 0; s0 < n_slices; s0 += 64) {              // slices in ascending groups of 64, fixed butterfly inside
    const int sl = s0 + lane;
    // (a slice without any probability has the maximum -inf and no sum of its own)
    tot += wave_sum(sl < n_slices && stat[sl].x != -INFINITY ? stat[sl].y * expf(stat[sl].x - m) : 0.f);
  }
  return make_float2(m, tot);
}
hipError_t launch_rows_softmax_stats(const float *logits, int rows, int vocab, float temp, float2 *part, hipStream_t st) {
  if (rows < 1 || vocab < 1 || !(temp > 0.f)) return hipErrorInvalidValue;
  const int n_slices = argmax_slices(vocab);
  hipLaunchKernelGGL(softmax_slice_kernel, dim3(n_slices, rows), dim3(kSelThreads), 0, st, logits, vocab, temp, n_slices, part);
  return hipGetLastError();
}

// ---- per-row top-k log-probabilities -------------------------------------------------------
// Stage 1: one workgroup per (slice of kTopkSlice entries, row): slice max, slice sum-exp and the
// slice's k best entries.  Each wavefront finds the k best of its own 1024 register-resident values by k
// rounds of a wave-wide argmax (shuffles only); the 4k finalists are then placed by rank.
// PER: values a thread holds, 16 for whole slices; vocabularies of up to 1024 tokens take 4 (a round goes through all of them, and so do maximum
// and sum: slices and merge of four rows of 1024, k = 4, 11.8 -> 10.2 us; same bits).
template <int PER>
__global__ __launch_bounds__(kSelThreads) void topk_slice_kernel(const float *logits, int vocab, int k, int n_slices,
                                                                 float *sc_val, int *sc_idx, float2 *sc_stat) {
  constexpr int NWV = kSelThreads / 64;
  __shared__ float shv[16];
  __shared__ float cv[NWV * kMaxTopK];
  __shared__ __attribute__((aligned(16))) uint64_t keys[NWV * kMaxTopK + 2];
  const int slice = blockIdx.x, rowi = blockIdx.y, t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int c0 = slice * kTopkSlice;
  const float *row = logits + (size_t)rowi * vocab;
  float v[PER];
#pragma unroll
  for (int e = 0; e < PER; e++) {
    const int c = c0 + t + e * kSelThreads;
    v[e] = c < vocab ? row[c] : -INFINITY;
  }
  float m = v[0];
#pragma unroll
  for (int e = 1; e < PER; e++) m = fmaxf(m, v[e]);
  m = block_max(m, shv);
  float s = 0.f;
#pragma unroll
  for (int e = 0; e < PER; e++) s += expf(v[e] - m);        // exp(-inf) = 0 for padding
  s = block_sum(s, shv);
  const size_t o = ((size_t)rowi * n_slices + slice);
  if (t == 0) sc_stat[o] = make_float2(m, s);
  uint32_t taken = 0;
  for (int r = 0; r < k; r++) {
    // best remaining value of the wave, then the lowest index carrying it
    float mv = -INFINITY;
#pragma unroll
    for (int e = 0; e < PER; e++) mv = fmaxf(mv, ((taken >> e) & 1u) ? -INFINITY : v[e]);
    const float best_v = wave_max_dpp(mv);
    int mi = INT_MAX;
#pragma unroll
    for (int e = PER - 1; e >= 0; e--) {
      const int c = c0 + t + e * kSelThreads;
      if (!((taken >> e) & 1u) && c < vocab && v[e] == best_v) mi = c;
    }
    const int best_i = wave_min_dpp(mi);
    if (lane == 0) { keys[wave * k + r] = order_key(best_v, best_i); cv[wave * k + r] = best_v; }
    if (best_i != INT_MAX && (best_i - c0) % kSelThreads == t) taken |= 1u << ((best_i - c0) / kSelThreads);
  }
  if (t < 2) keys[NWV * k + t] = 0ull;                       // padding for the pairwise reads
  __syncthreads();
  if (t < NWV * k) {
    const uint64_t key = keys[t];
    const int rank = key_rank(keys, (NWV * k + 1) & ~1, key, t);
    if (rank < k) {
      const bool valid = key != 0ull;
      sc_val[o * kMaxTopK + rank] = valid ? cv[t] : -INFINITY;
      sc_idx[o * kMaxTopK + rank] = valid ? 0x7FFFFFFF - (int)(uint32_t)key : INT_MAX;
    }
  }
}
// Stage 2: one workgroup of two wavefronts per row.  The first merges the slices' lists, which are sorted: every lane holds the best entry not yet
// taken of its lists, each of the k rounds takes the best of all lanes and the lane it came from moves on.  The second forms the row's
// log-sum-exp meanwhile.  (Ranking every candidate against every other one took 20 us at 32 slices of 10 where this takes 6.)
// FEW: up to 64 slices, one per lane and whole in its registers; else lane l walks the slices l, l + 64, .. in the LDS.
constexpr int kMaxMergeCand = 4096;
constexpr int kMergeThreads = 128;
// The k best of up to 64 sorted lists (lane sl: slice sl's, whole in its registers), by one wavefront: best(r, value, index) for r = 0 .. k - 1, in lane 0.
template <typename Best>
__device__ __forceinline__ void merge_lists(int k, int n_slices, const float *val, const int *idx, int lane, Best best) {
  float v[kMaxTopK];
  int i[kMaxTopK];
  const int sl = min(lane, n_slices - 1);
#pragma unroll
  for (int r = 0; r < kMaxTopK; r++) { v[r] = val[sl * kMaxTopK + min(r, k - 1)]; i[r] = idx[sl * kMaxTopK + min(r, k - 1)]; }
#pragma unroll
  for (int r = 0; r < kMaxTopK; r++)
    if (lane >= n_slices || r >= k) { v[r] = -INFINITY; i[r] = INT_MAX; }
  for (int r = 0; r < k; r++) {
    const float bv = wave_max_dpp(v[0]);
    const int bi = wave_min_dpp(v[0] == bv ? i[0] : INT_MAX);
    if (lane == 0) best(r, bv, bi);
    if (i[0] != bi || bi == INT_MAX) continue;                // (a token is in one list only)
#pragma unroll
    for (int e = 0; e + 1 < kMaxTopK; e++) { v[e] = v[e + 1]; i[e] = i[e + 1]; }
    v[kMaxTopK - 1] = -INFINITY; i[kMaxTopK - 1] = INT_MAX;
  }
}
// log-sum-exp of a row from its slices' statistics, by one wavefront
__device__ __forceinline__ float lists_lse(int n_slices, const float2 *stat, int lane) {
  float m = -INFINITY;
  for (int sl = lane; sl < n_slices; sl += 64) m = fmaxf(m, stat[sl].x);
  m = wave_max(m);
  float tot = 0.f;
  for (int s0 = 0; s0 < n_slices; s0 += 64) {                // slices in ascending groups of 64, fixed butterfly inside
    const int sl = s0 + lane;
    // (a slice without any probability has the maximum -inf and no sum of its own)
    tot += wave_sum(sl < n_slices && stat[sl].x != -INFINITY ? stat[sl].y * expf(stat[sl].x - m) : 0.f);
  }
  return m + logf(tot);
}
template <bool FEW>
__global__ __launch_bounds__(kMergeThreads) void topk_merge_kernel(int k, int n_slices, const float *sc_val, const int *sc_idx,
                                                                   const float2 *sc_stat, int *top_tok, float *top_lp) {
  __shared__ float cand_val[FEW ? 1 : kMaxMergeCand];
  __shared__ int cand_idx[FEW ? 1 : kMaxMergeCand];
  __shared__ uint8_t taken[FEW ? 1 : kMaxMergeCand];          // of each slice's list
  __shared__ float lse_sh, best_val[kMaxTopK];
  __shared__ int best_idx[kMaxTopK];
  const int rowi = blockIdx.x, t = threadIdx.x, lane = t & 63;
  const float *val = sc_val + (size_t)rowi * n_slices * kMaxTopK;
  const int *idx = sc_idx + (size_t)rowi * n_slices * kMaxTopK;
  auto best = [&](int r, float v, int i) __attribute__((always_inline)) { best_val[r] = v; best_idx[r] = i; };
  if constexpr (!FEW) {
    for (int id = t; id < n_slices * k; id += kMergeThreads) {   // candidate id = slice * k + r
      const int at = id / k * kMaxTopK + id % k;
      cand_val[id] = val[at]; cand_idx[id] = idx[at];
    }
    for (int sl = t; sl < n_slices; sl += kMergeThreads) taken[sl] = 0;
    __syncthreads();
  }
  if (t < 64) {
    if constexpr (FEW) {
      merge_lists(k, n_slices, val, idx, lane, best);
    } else {
      float v;                                                // the best entry left in this lane's lists
      int i, from;
      auto head = [&]() __attribute__((always_inline)) {
        v = -INFINITY; i = INT_MAX; from = -1;
        for (int sl = lane; sl < n_slices; sl += 64) {
          const int r = taken[sl];
          if (r >= k) continue;
          const float x = cand_val[sl * k + r];
          const int c = cand_idx[sl * k + r];
          if (c != INT_MAX && (from < 0 || better(x, c, v, i))) { v = x; i = c; from = sl; }
        }
      };
      head();
      for (int r = 0; r < k; r++) {
        const float bv = wave_max_dpp(v);
        const int bi = wave_min_dpp(v == bv ? i : INT_MAX);
        if (lane == 0) best(r, bv, bi);
        if (i != bi || bi == INT_MAX) continue;               // (a token is in one list only)
        taken[from]++;
        head();
      }
    }
  } else {
    const float lse = lists_lse(n_slices, sc_stat + (size_t)rowi * n_slices, lane);
    if (lane == 0) lse_sh = lse;
  }
  __syncthreads();
  if (t < k) {
    top_tok[rowi * kMaxTopK + t] = best_idx[t];
    top_lp[rowi * kMaxTopK + t] = best_val[t] - lse_sh;
  }
}
static hipError_t launch_topk_slices(const float *logits, int rows, int vocab, int k, float *sc_val, int *sc_idx, float2 *sc_stat, hipStream_t st) {
  const int n_slices = (vocab + kTopkSlice - 1) / kTopkSlice;
  if (rows < 1 || k < 1 || k > kMaxTopK || k > vocab || n_slices * k > kMaxMergeCand) return hipErrorInvalidValue;
  const auto kernel = vocab <= 4 * kSelThreads ? topk_slice_kernel<4> : topk_slice_kernel<kTopkSlice / kSelThreads>;
  hipLaunchKernelGGL(kernel, dim3(n_slices, rows), dim3(kSelThreads), 0, st, logits, vocab, k, n_slices, sc_val, sc_idx, sc_stat);
  return hipGetLastError();
}
hipError_t launch_rows_topk_logprob(const float *logits, int rows, int vocab, int k, float *sc_val, int *sc_idx,
                                    float2 *sc_stat, int *top_tok, float *top_lp, hipStream_t st) {
  const int n_slices = (vocab + kTopkSlice - 1) / kTopkSlice;
  const hipError_t e = launch_topk_slices(logits, rows, vocab, k, sc_val, sc_idx, sc_stat, st);
  if (e != hipSuccess) return e;
  if (n_slices <= 64)
    hipLaunchKernelGGL(topk_merge_kernel<true>, dim3(rows), dim3(kMergeThreads), 0, st, k, n_slices, sc_val, sc_idx, sc_stat, top_tok, top_lp);
  else
    hipLaunchKernelGGL(topk_merge_kernel<false>, dim3(rows), dim3(kMergeThreads), 0, st, k, n_slices, sc_val, sc_idx, sc_stat, top_tok, top_lp);
  return hipGetLastError();
}

// ---- candidate pool ------------------------------------------------------------------------
// One workgroup: wavefront r merges the slices' lists of row r and forms its log-sum-exp (the same as topk_merge_kernel, bit for bit), then the pool takes
// the rows' children.  Merge and pool were two launches of one workgroup's work each, a chain per draft depth: root step and five expansions at the
// 7B shape 12 launches -> 6.
constexpr int kPoolThreads = kMaxTopK * 64;
struct TopRows { const float *sc_val; const int *sc_idx; const float2 *sc_stat; int n_slices; const int *tok; const float *lp; };   // tok: merged already (more than 64 slices)
struct TopShared { int tok[kMaxTopK * kMaxTopK]; float lp[kMaxTopK * kMaxTopK]; };
__device__ __forceinline__ void merge_rows(const TopRows &top, int rows, int k, TopShared &sh) {
  const int lane = threadIdx.x & 63, r = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (top.tok != nullptr) {
    if (r < rows && lane < k) { sh.tok[r * kMaxTopK + lane] = top.tok[r * kMaxTopK + lane]; sh.lp[r * kMaxTopK + lane] = top.lp[r * kMaxTopK + lane]; }
  } else if (r < rows) {
    const size_t at = (size_t)r * top.n_slices;
    const float lse = lists_lse(top.n_slices, top.sc_stat + at, lane);
    merge_lists(k, top.n_slices, top.sc_val + at * kMaxTopK, top.sc_idx + at * kMaxTopK, lane,
                [&](int j, float v, int i) __attribute__((always_inline)) { sh.tok[r * kMaxTopK + j] = i; sh.lp[r * kMaxTopK + j] = v - lse; });
  }
  __syncthreads();
}
__global__ __launch_bounds__(64) void pool_init_kernel(DraftState s, TopRows top, int k, int root_row, const int *n_draft_ptr) {
  __shared__ TopShared sh;
  const int r = threadIdx.x;
  const int n_draft = *n_draft_ptr;
  merge_rows(top, 1, k, sh);
  if (r < k) {
    s.pool_tok[r] = sh.tok[r]; s.pool_par[r] = -1; s.pool_dep[r] = 1; s.pool_sc[r] = sh.lp[r];
    s.front_pool[r] = r; s.front_tok[r] = sh.tok[r]; s.front_src[r] = root_row; s.front_depth[r] = 0;
    s.front_anc[r * kAncStride] = r;
    s.front_slot[r] = n_draft + r;
    s.front_pos[r] = n_draft + 1;
  }
  if (r == 0) *s.n_pool = k;
}
// `step` t in 2..D: the k frontier rows are nodes of depth t-1; their children have depth t.
__global__ __launch_bounds__(kPoolThreads) void pool_expand_kernel(DraftState s, TopRows top, int k, int step, const int *n_draft_ptr, int select_next) {
  __shared__ TopShared sh;
  __shared__ float sc[kMaxTopK * kMaxTopK];
  __shared__ int old_anc[kMaxTopK * kAncStride];
  __shared__ int old_pool[kMaxTopK];
  __shared__ float old_sc[kMaxTopK];
  const int t = threadIdx.x, kk = k * k;
  const int n_draft = *n_draft_ptr;
  const int base = *s.n_pool;
  if (t < k) { const int p = s.front_pool[t]; old_pool[t] = p; old_sc[t] = s.pool_sc[p]; }
  if (t < k * kAncStride) old_anc[t] = s.front_anc[t];
  merge_rows(top, k, k, sh);
  int r = 0, j = 0, tok = 0;
  if (t < kk) {
    r = t / k; j = t % k;                                   // children in (frontier order, best first) order
    tok = sh.tok[r * kMaxTopK + j];
    const float v = old_sc[r] + sh.lp[r * kMaxTopK + j];
    sc[t] = v;
    s.pool_tok[base + t] = tok; s.pool_par[base + t] = old_pool[r]; s.pool_dep[base + t] = step; s.pool_sc[base + t] = v;
  }
  __syncthreads();
  if (t == 0) *s.n_pool = base + kk;
  if (!select_next || t >= kk) return;
  int rank = 0;
  for (int c = 0; c < kk; c++) rank += better(sc[c], c, sc[t], t) ? 1 : 0;
  if (rank >= k) return;
  // this child is row `rank` of the next expansion step (step + 1): depth argument step - 1
  s.front_pool[rank] = base + t; s.front_tok[rank] = tok; s.front_src[rank] = r; s.front_depth[rank] = step - 1;
  for (int a = 0; a < step - 1; a++) s.front_anc[rank * kAncStride + a] = old_anc[r * kAncStride + a];
  s.front_anc[rank * kAncStride + step - 1] = (step - 1) * k + rank;
  s.front_slot[rank] = n_draft + (step - 1) * k + rank;
  s.front_pos[rank] = n_draft + 1 + (step - 1);
}
static_assert(kMaxTopK * kAncStride <= kMaxTopK * 64, "a thread per ancestor entry");
// The rows' slices, merged by the kernel that follows; of a vocabulary of more than 64 slices by a launch of their own.
static hipError_t top_rows(const float *logits, int rows, int vocab, int k, float *sc_val, int *sc_idx, float2 *sc_stat, int *top_tok, float *top_lp,
                           TopRows *top, hipStream_t st) {
  const int n_slices = (vocab + kTopkSlice - 1) / kTopkSlice;
  const bool few = n_slices <= 64;
  *top = TopRows{sc_val, sc_idx, sc_stat, n_slices, few ? nullptr : top_tok, top_lp};
  return few ? launch_topk_slices(logits, rows, vocab, k, sc_val, sc_idx, sc_stat, st)
             : launch_rows_topk_logprob(logits, rows, vocab, k, sc_val, sc_idx, sc_stat, top_tok, top_lp, st);
}
hipError_t launch_pool_init(const DraftState &s, const float *logits, int vocab, float *sc_val, int *sc_idx, float2 *sc_stat, int *top_tok, float *top_lp,
                            int k, int root_row, const int *n_draft, hipStream_t st) {
  TopRows top;
  const hipError_t e = top_rows(logits, 1, vocab, k, sc_val, sc_idx, sc_stat, top_tok, top_lp, &top, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(pool_init_kernel, dim3(1), dim3(64), 0, st, s, top, k, root_row, n_draft);
  return hipGetLastError();
}
hipError_t launch_pool_expand(const DraftState &s, const float *logits, int vocab, float *sc_val, int *sc_idx, float2 *sc_stat, int *top_tok, float *top_lp,
                              int k, int step, const int *n_draft, int select_next, hipStream_t st) {
  if (step < 2 || step > kMaxDepth) return hipErrorInvalidValue;
  TopRows top;
  const hipError_t e = top_rows(logits, k, vocab, k, sc_val, sc_idx, sc_stat, top_tok, top_lp, &top, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(pool_expand_kernel, dim3(1), dim3(k * 64), 0, st, s, top, k, step, n_draft, select_next);
  return hipGetLastError();
}

// ---- rerank --------------------------------------------------------------------------------
constexpr int kMaxPool = kMaxTopK + (kMaxDepth - 1) * kMaxTopK * kMaxTopK;    // 3600
constexpr int kPoolWords = (kMaxPool + 31) / 32;
constexpr int kRerankThreads = 1024;
__global__ __launch_bounds__(kRerankThreads) void rerank_kernel(DraftState s, int total, const int *root_tok, int *tree_n,
                                                                int *tree_tok, int *tree_par, int *tree_dep, float *tree_sc) {
  typedef __attribute__((ext_vector_type(4))) float f32x4_t;
  __shared__ __attribute__((aligned(16))) float sc[kMaxPool + 4];
  __shared__ uint32_t kept[kPoolWords];                     // bit c: pool entry c is in the tree
  __shared__ int before[kPoolWords];                        // kept entries in earlier words
  const int t = threadIdx.x, n = *s.n_pool;
  const int keep = min(total - 1, n);
  const int n_words = (n + 31) / 32, n4 = (n + 3) & ~3;
  for (int c = t; c < n4; c += kRerankThreads) sc[c] = c < n ? s.pool_sc[c] + 0.f : -INFINITY;
  for (int w = t; w < n_words; w += kRerankThreads) kept[w] = 0u;
  __syncthreads();
  for (int c = t; c < n; c += kRerankThreads) {
    // rank = entries with a larger score, plus equal scores at a lower pool index
    const float v = sc[c];
    int rank = 0;
#pragma unroll 2
    for (int o = 0; o < n4; o += 4) {
      const f32x4_t x = *(const f32x4_t *)(sc + o);
      rank += (x.x > v || (x.x == v && o < c)) ? 1 : 0;
      rank += (x.y > v || (x.y == v && o + 1 < c)) ? 1 : 0;
      rank += (x.z > v || (x.z == v && o + 2 < c)) ? 1 : 0;
      rank += (x.w > v || (x.w == v && o + 3 < c)) ? 1 : 0;
    }
    if (rank < keep) atomicOr(&kept[c >> 5], 1u << (c & 31));
  }
  __syncthreads();
  for (int w = t; w < n_words; w += kRerankThreads) {
    int cnt = 0;
    for (int u = 0; u < w; u++) cnt += __popc(kept[u]);
    before[w] = cnt;
  }
  __syncthreads();
  // node index = 1 + number of kept entries with a lower pool index (kept in pool order: parents first)
  auto node_of = [&](int c) { return 1 + before[c >> 5] + __popc(kept[c >> 5] & ((1u << (c & 31)) - 1u)); };
  for (int c = t; c < n; c += kRerankThreads) {
    if (!((kept[c >> 5] >> (c & 31)) & 1u)) continue;
    const int j = node_of(c);
    const int par = s.pool_par[c];
    tree_tok[j] = s.pool_tok[c];
    tree_par[j] = par < 0 ? 0 : node_of(par);               // a parent outscores (or ties at a lower index) its children, so it is kept
    tree_dep[j] = s.pool_dep[c];
    tree_sc[j] = s.pool_sc[c];
  }
  if (t == 0) { tree_tok[0] = *root_tok; tree_par[0] = -1; tree_dep[0] = 0; tree_sc[0] = 0.f; *tree_n = keep + 1; }
}
hipError_t launch_rerank(const DraftState &s, int total, const int *root_tok, int *tree_n, int *tree_tok, int *tree_par,
                         int *tree_dep, float *tree_sc, hipStream_t st) {
  if (total < 1 || total > kMaxNodes) return hipErrorInvalidValue;
  hipLaunchKernelGGL(rerank_kernel, dim3(1), dim3(kRerankThreads), 0, st, s, total, root_tok, tree_n, tree_tok, tree_par, tree_dep,
                     tree_sc);
  return hipGetLastError();
}

// ---- acceptance ----------------------------------------------------------------------------
// f(v, load(v)) for the thread's share v = threadIdx.x, + blockDim.x, ... of [0, n) in ascending order, with the loads of U
// entries in flight (one workgroup walks a whole vocabulary row: taken one by one, every entry waits for its own load).
template <int U = 8, typename Load, typename F>
__device__ __forceinline__ void for_share(int n, Load load, F f) {
  const int T = blockDim.x;
  if (n <= 2 * T) {                                           // too short a share to fill the loads: 1000 entries 37.4 us with them (five nodes), 35.6 without
    for (int v = threadIdx.x; v < n; v += T) f(v, load(v));
    return;
  }
  for (int v0 = threadIdx.x; v0 < n; v0 += U * T) {
    decltype(load(0)) x[U];
#pragma unroll
    for (int u = 0; u < U; u++) x[u] = load(min(v0 + u * T, n - 1));
#pragma unroll
    for (int u = 0; u < U; u++)
      if (v0 + u * T < n) f(v0 + u * T, x[u]);
  }
}

// Gumbel-max over one row, skipping `n_rem` removed tokens.  Whole block; result to every thread.
__device__ __forceinline__ int gumbel_argmax(const float *row, int vocab, float temp, uint64_t stream, const int *rem,
                                             int n_rem, float *shv, int *shi) {
  ValIdx b{-INFINITY, INT_MAX};
  for_share(vocab, [&](int v) { return row[v]; }, [&](int v, float x) {
    bool skip = false;
    for (int r = 0; r < n_rem; r++) skip |= rem[r] == v;
    const float z = x / temp + rng_gumbel(stream, v);
    if (!skip && (z > b.v || b.i == INT_MAX)) { b.v = z; b.i = v; }
  });
  return block_best(b, shv, shi).i;
}

// The children of node `cur` in node order, by the first wavefront from the parents in LDS -> kid[0 .. return value).
__device__ __forceinline__ int list_children(const int *par, int n_nodes, int cur, int lane, int *kid) {
  int n = 0;
#pragma unroll
  for (int c0 = 0; c0 < kMaxNodes; c0 += 64) {
    const int c = c0 + lane;
    const bool is = c > cur && c < n_nodes && par[c] == cur;
    const uint64_t mask = __ballot(is);
    if (is) kid[n + __popcll(mask & ((1ull << lane) - 1ull))] = c;
    n += __popcll(mask);
  }
  return n;
}

// Multi-round rejection sampling down the tree.  The children of a node were chosen
// deterministically by the draft (top-k), so each is a point-mass proposal: child c is accepted
// with probability p'(c), where p' is the target distribution with the already rejected siblings
// removed and renormalised; when all children are rejected the bonus token is drawn from p'.
// One workgroup.  Per visited node: the first wavefront merges the row's softmax slices and lists the
// node's children, all threads fetch the children's logits together, thread 0 runs the (inherently
// sequential) accept/reject chain on those values, and the bonus draw uses the whole workgroup.
constexpr int kAcceptThreads = 1024;
__global__ __launch_bounds__(kAcceptThreads) void accept_sample_kernel(const float *logits, int vocab, const float2 *stat_part,
                                                                       int n_slices, float temp, const int *tree_tok,
                                                                       const int *tree_par, int n_nodes, uint64_t seed,
                                                                       uint32_t cycle, AcceptResult *res) {
  __shared__ float shv[16];
  __shared__ int shi[16];
  __shared__ int rem[kMaxNodes];
  __shared__ int kid[kMaxNodes], par[kMaxNodes];
  __shared__ float kid_x[kMaxNodes];
  __shared__ int sh_next, sh_nrem, sh_nkid;
  __shared__ float2 sh_stat;
  const int t = threadIdx.x;
  int cur = 0, m = 0;
  if (t == 0) res->node[0] = 0;
  if (t < n_nodes) par[t] = tree_par[t];
  __syncthreads();
  for (int step = 0; step <= kMaxDepth; step++) {
    const uint64_t stream = rng_stream(seed, cycle, (uint32_t)cur);
    const float *row = logits + (size_t)cur * vocab;
    if (t < 64) {
      const float2 st = merge_softmax_stats(stat_part, n_slices, cur, t);
      const int nk = m < kMaxDepth ? list_children(par, n_nodes, cur, t, kid) : 0;   // node order = descending draft probability
      if (t == 0) { sh_stat = st; sh_nkid = nk; }
    }
    __syncthreads();
    const int n_kid = sh_nkid;
    if (t < n_kid) kid_x[t] = row[tree_tok[kid[t]]];
    __syncthreads();
    if (t == 0) {
      const float2 st = sh_stat;
      float removed = 0.f;                                  // probability mass of the rejected siblings
      int n_rem = 0, next = -1;
      for (int ord = 0; ord < n_kid && next < 0; ord++) {
        const int c = kid[ord];
        const int tok = tree_tok[c];
        bool dup = false;
        for (int r = 0; r < n_rem; r++) dup |= rem[r] == tok;
        const float p0 = dup ? 0.f : expf(kid_x[ord] / temp - st.x) / st.y;
        const float rest = 1.0f - removed;
        const float u = rng_uniform(stream, (uint64_t)ord);
        if (u < p0 / rest) { next = c; break; }
        if (!dup) { removed += p0; rem[n_rem++] = tok; }
        if (!(1.0f - removed > 0.f)) { next = c; break; }   // nothing left in the residual: c was certain
      }
      sh_next = next; sh_nrem = n_rem;
    }
    __syncthreads();
    const int next = sh_next, n_rem = sh_nrem;
    if (next >= 0) {
      if (t == 0) { res->token[m] = tree_tok[next]; res->node[m + 1] = next; }
      cur = next; m++;
      __syncthreads();
      continue;
    }
    const int bonus = gumbel_argmax(row, vocab, temp, stream, rem, n_rem, shv, shi);
    if (t == 0) res->token[m] = bonus;
    break;
  }
  if (t == 0) res->n_acc = m;
}
hipError_t launch_accept_sample(const float *logits, int vocab, const float2 *stat_part, float temp, const int *tree_tok,
                                const int *tree_par, int n_nodes, uint64_t seed, uint32_t cycle, AcceptResult *res,
                                hipStream_t st) {
  if (n_nodes < 1 || n_nodes > kMaxNodes || !(temp > 0.f)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(accept_sample_kernel, dim3(1), dim3(kAcceptThreads), 0, st, logits, vocab, stat_part, argmax_slices(vocab),
                     temp, tree_tok, tree_par, n_nodes, seed, cycle, res);
  return hipGetLastError();
}

// The ratio rule for SAMPLED children (the textbook speculative-sampling acceptance, Sec. 2 third step): at
// node `cur` with target distribution p and draft distribution q (both softmax(row / temp)), the children,
// drawn from q without replacement and tried in node order, are accepted with probability min(1, p_j / q_j);
// a rejection replaces p by normalise(max(p - q, 0)) and removes the child from q; when every child is
// rejected the next token is drawn from the current p (Gumbel-max).  One workgroup.  Until the first rejection at a
// node p and q are needed at the children's tokens only: with the rows' softmax statistics at hand (p_stat by node,
// q_stat by draft row: {max, sum exp} per slice; nullptr: both are computed here) an accepted node costs no pass over the
// vocabulary.  After a rejection the current p lives in `work` (vocab floats, unnormalised, with its normaliser in a
// register); a thread only ever re-reads the entries it wrote itself, and the entry of a child's token is handed to the
// others through LDS.  26 nodes, vocabulary 128256, five to six accepted: 716 -> 95 us, and 2 x 6 for the statistics.
__global__ __launch_bounds__(kAcceptThreads) void accept_qratio_kernel(const float *p_logits, const float *q_logits,
                                                                       const int *qrow_of, const float2 *p_stat, const float2 *q_stat,
                                                                       int n_slices, int vocab, float temp,
                                                                       const int *tree_tok, const int *tree_par, int n_nodes,
                                                                       uint64_t seed, uint32_t cycle, float *work,
                                                                       AcceptResult *res) {
  __shared__ float shv[16];
  __shared__ int shi[16];
  __shared__ int rem[kMaxNodes];
  __shared__ int kid[kMaxNodes], par[kMaxNodes];
  __shared__ int sh_nkid;
  __shared__ float sh_px, sh_q0;
  __shared__ float2 sh_p, sh_q;
  const int t = threadIdx.x;
  int cur = 0, m = 0;
  if (t == 0) res->node[0] = 0;
  if (t < n_nodes) par[t] = tree_par[t];
  __syncthreads();
  for (int step = 0; step <= kMaxDepth; step++) {
    const uint64_t stream = rng_stream(seed, cycle, (uint32_t)cur);
    if (t < 64) {
      const int nk = m < kMaxDepth ? list_children(par, n_nodes, cur, t, kid) : 0;   // node order = draw order
      if (t == 0) sh_nkid = nk;
    }
    __syncthreads();
    const int n_kid = sh_nkid;
    const float *prow = p_logits + (size_t)cur * vocab;
    // the draft row of a node without children is never read (it may not exist: qrow_of[cur] < 0)
    const int qr = n_kid == 0 ? 0 : (qrow_of ? qrow_of[cur] : cur);
    const float *qrow = n_kid == 0 ? prow : q_logits + (size_t)qr * vocab;
    float mp = -INFINITY, mq = -INFINITY, sp = 0.f, sq = 0.f;
    if (p_stat != nullptr) {
      if (t < 64) {
        const float2 st = merge_softmax_stats(p_stat, n_slices, cur, t);
        if (t == 0) sh_p = st;
      } else if (t < 128 && n_kid > 0) {
        const float2 st = merge_softmax_stats(q_stat, n_slices, qr, t - 64);
        if (t == 64) sh_q = st;
      }
      __syncthreads();
      mp = sh_p.x; sp = sh_p.y;
      if (n_kid > 0) { mq = sh_q.x; sq = sh_q.y; }
    } else {
      auto both = [&](int v) { return make_float2(prow[v], qrow[v]); };
      for_share(vocab, both, [&](int, float2 x) { mp = fmaxf(mp, x.x / temp); mq = fmaxf(mq, x.y / temp); });
      mp = block_max(mp, shv);
      mq = block_max(mq, shv);
      for_share(vocab, both, [&](int, float2 x) { sp += expf(x.x / temp - mp); sq += expf(x.y / temp - mq); });
      sp = block_sum(sp, shv);
      sq = block_sum(sq, shv);
    }
    bool in_work = false;                                     // p(v) = work[v] * inv_zp, before the first rejection exp(..) * inv_zp
    float inv_zp = 1.f / sp;
    float removed = 0.f, inv_zq = 1.f;                        // q_j(v) = q(v) * inv_zq for v not removed, else 0
    int next = -1, n_rem = 0;
    for (int ord = 0; ord < n_kid && next < 0; ord++) {
      const int c = kid[ord];
      const int x = tree_tok[c];
      bool dup = false;
      for (int r = 0; r < n_rem; r++) dup |= rem[r] == x;
      if (x % kAcceptThreads == t) {
        sh_px = (in_work ? work[x] : expf(prow[x] / temp - mp)) * inv_zp;
        sh_q0 = expf(qrow[x] / temp - mq) / sq;
      }
      __syncthreads();
      const float px = sh_px, q0 = dup ? 0.f : sh_q0;
      const float u = rng_uniform(stream, (uint64_t)ord);
      if (u * (q0 * inv_zq) < px) { next = c; break; }
      // rejected: p <- max(p - q_j, 0), renormalised; q_{j+1} <- q_j without x
      float part = 0.f;
      for_share(vocab, [&](int v) { return make_float2(in_work ? work[v] : prow[v], qrow[v]); }, [&](int v, float2 y) {
        bool gone = false;
        for (int r = 0; r < n_rem; r++) gone |= rem[r] == v;
        const float qv = gone ? 0.f : expf(y.y / temp - mq) / sq * inv_zq;
        const float nv = fmaxf((in_work ? y.x : expf(y.x / temp - mp)) * inv_zp - qv, 0.f);
        work[v] = nv;
        part += nv;
      });
      in_work = true;
      const float zp = block_sum(part, shv);                  // (its barriers also order the LDS traffic of this round)
      if (!(zp > 0.f)) { next = c; break; }                   // nothing left in the residual: c was certain
      inv_zp = 1.f / zp;
      if (!dup) {
        if (t == 0) rem[n_rem] = x;
        n_rem++;
        removed += q0;
        inv_zq = 1.f - removed > 0.f ? 1.f / (1.f - removed) : 0.f;
      }
      __syncthreads();
    }
    if (next >= 0) {
      if (t == 0) { res->token[m] = tree_tok[next]; res->node[m + 1] = next; }
      cur = next; m++;
      __syncthreads();
      continue;
    }
    ValIdx b{-INFINITY, INT_MAX};
    for_share(vocab, [&](int v) { return in_work ? work[v] : prow[v]; }, [&](int v, float y) {
      const float pv = (in_work ? y : expf(y / temp - mp)) * inv_zp;
      const float z = logf(pv) + rng_gumbel(stream, v);
      if (pv > 0.f && (z > b.v || b.i == INT_MAX)) { b.v = z; b.i = v; }
    });
    const int bonus = block_best(b, shv, shi).i;
    if (t == 0) res->token[m] = bonus;
    break;
  }
  if (t == 0) res->n_acc = m;
}
hipError_t launch_accept_qratio(const float *p_logits, const float *q_logits, const int *qrow_of, const float2 *p_stat, const float2 *q_stat,
                                int vocab, float temp, const int *tree_tok, const int *tree_par, int n_nodes, uint64_t seed,
                                uint32_t cycle, float *work, AcceptResult *res, hipStream_t st) {
  if (n_nodes < 1 || n_nodes > kMaxNodes || vocab < 1 || !(temp > 0.f)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(accept_qratio_kernel, dim3(1), dim3(kAcceptThreads), 0, st, p_logits, q_logits, qrow_of, p_stat, q_stat,
                     argmax_slices(vocab), vocab, temp, tree_tok, tree_par, n_nodes, seed, cycle, work, res);
  return hipGetLastError();
}

// ---- static tree shapes ----------------------------------------------------------------------
// After the proposals of the nodes of depth d-1 are known (top_tok / top_lp, row = the node's row in its
// depth's forward, 0 for the root): fill token / parent / depth / score of the nodes of depth d, and for those
// of them that have children set up their row of the next draft forward (the same tables the dynamic
// expansion builds: token, source row of the parent's predicted feature, depth argument, ancestor slots).
__global__ void static_step_kernel(StaticTables tb, int d, const int *top_tok, const float *top_lp, int root_row,
                                   const int *root_tok, const int *n_draft_ptr, int with_scores, DraftState s, int *t_n,
                                   int *t_tok, int *t_par, int *t_dep, float *t_sc) {
  const int i = threadIdx.x;
  const int n_draft = *n_draft_ptr;
  if (i == 0 && d == 1) { *t_n = tb.n_nodes; t_tok[0] = *root_tok; t_par[0] = -1; t_dep[0] = 0; t_sc[0] = 0.f; }
  if (i < 1 || i >= tb.n_nodes || tb.depth[i] != d) return;
  const int p = tb.parent[i];
  const int pr = d == 1 ? 0 : tb.erow[p];
  const int tok = top_tok[pr * kMaxTopK + tb.rank[i]];
  t_tok[i] = tok; t_par[i] = p; t_dep[i] = d;
  t_sc[i] = with_scores ? (d == 1 ? 0.f : t_sc[p]) + top_lp[pr * kMaxTopK + tb.rank[i]] : 0.f;
  const int r = tb.erow[i];
  if (r < 0) return;
  s.front_tok[r] = tok;
  s.front_src[r] = d == 1 ? root_row : tb.erow[p];
  s.front_depth[r] = d - 1;
  s.front_slot[r] = n_draft + tb.eoff[i];
  s.front_pos[r] = n_draft + d;
  for (int a = i, q = d - 1; q >= 0; q--, a = tb.parent[a]) s.front_anc[r * kAncStride + q] = tb.eoff[a];
}
hipError_t launch_static_step(const StaticTables &tb, int d, const int *top_tok, const float *top_lp, int root_row,
                              const int *root_tok, const int *n_draft, int with_scores, const DraftState &s, int *t_n, int *t_tok,
                              int *t_par, int *t_dep, float *t_sc, hipStream_t st) {
  if (tb.n_nodes < 1 || tb.n_nodes > kMaxNodes || d < 1 || d > kMaxDepth) return hipErrorInvalidValue;
  hipLaunchKernelGGL(static_step_kernel, dim3(1), dim3(kMaxNodes), 0, st, tb, d, top_tok, top_lp, root_row, root_tok, n_draft,
                     with_scores, s, t_n, t_tok, t_par, t_dep, t_sc);
  return hipGetLastError();
}

// z[r][v] = logits[r][v] / temp + Gumbel noise of stream (seed, cycle, node_stream[r]) for rows r < rows.
__global__ __launch_bounds__(kSelThreads) void perturb_rows_kernel(const float *logits, int vocab, float temp, uint64_t seed,
                                                                   uint32_t cycle, const int *node_stream, float *z) {
  const int r = blockIdx.y;
  const uint64_t stream = rng_stream(seed, cycle, (uint32_t)node_stream[r]);
  const float *row = logits + (size_t)r * vocab;
  float *zr = z + (size_t)r * vocab;
  for (int v = blockIdx.x * kSelThreads + threadIdx.x; v < vocab; v += gridDim.x * kSelThreads)
    zr[v] = row[v] / temp + rng_gumbel(stream, v);
}
hipError_t launch_perturb_rows(const float *logits, int rows, int vocab, float temp, uint64_t seed, uint32_t cycle,
                               const int *node_stream, float *z, hipStream_t st) {
  if (rows < 1 || rows > kMaxTopK || vocab < 1 || !(temp > 0.f)) return hipErrorInvalidValue;
  const int blocks = (vocab + kSelThreads - 1) / kSelThreads;
  hipLaunchKernelGGL(perturb_rows_kernel, dim3(blocks > 256 ? 256 : blocks, rows), dim3(kSelThreads), 0, st, logits, vocab, temp, seed,
                     cycle, node_stream, z);
  return hipGetLastError();
}

// out[i] = the i-th of m tokens drawn without replacement from softmax(logits / temp): the m largest of
// logits / temp + Gumbel noise of stream (seed, cycle, node), found by the two-stage top-k above on the
// perturbed row (written to `z`, vocab floats).
__global__ __launch_bounds__(kSelThreads) void perturb_gumbel_kernel(const float *logits, int vocab, float temp, uint64_t seed,
                                                                     uint32_t cycle, uint32_t node, float *z) {
  const uint64_t stream = rng_stream(seed, cycle, node);
  for (int v = blockIdx.x * kSelThreads + threadIdx.x; v < vocab; v += gridDim.x * kSelThreads)
    z[v] = logits[v] / temp + rng_gumbel(stream, v);
}
__global__ void copy_ints_kernel(const int *src, int n, int *dst) {
  if ((int)threadIdx.x < n) dst[threadIdx.x] = src[threadIdx.x];
}
hipError_t launch_sample_children(const float *logits, int vocab, float temp, int m, uint64_t seed, uint32_t cycle, uint32_t node,
                                  float *z, float *sc_val, int *sc_idx, float2 *sc_stat, int *top_tok, float *top_lp, int *out,
                                  hipStream_t st) {
  if (vocab < 1 || m < 1 || m > kMaxTopK || m > vocab || !(temp > 0.f)) return hipErrorInvalidValue;
  const int blocks = (vocab + kSelThreads - 1) / kSelThreads;
  hipLaunchKernelGGL(perturb_gumbel_kernel, dim3(blocks > 1024 ? 1024 : blocks), dim3(kSelThreads), 0, st, logits, vocab, temp, seed,
                     cycle, node, z);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = launch_rows_topk_logprob(z, 1, vocab, m, sc_val, sc_idx, sc_stat, top_tok, top_lp, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(copy_ints_kernel, dim3(1), dim3(64), 0, st, top_tok, m, out);
  return hipGetLastError();
}

__global__ __launch_bounds__(kAcceptThreads) void sample_row_kernel(const float *logits, int vocab, float temp, uint64_t seed,
                                                                    uint32_t cycle, uint32_t node, int *out) {
  __shared__ float shv[16];
  __shared__ int shi[16];
  const int tok = gumbel_argmax(logits, vocab, temp, rng_stream(seed, cycle, node), nullptr, 0, shv, shi);
  if (threadIdx.x == 0) *out = tok;
}
hipError_t launch_sample_row(const float *logits, int vocab, float temp, uint64_t seed, uint32_t cycle, uint32_t node,
                             int *out, hipStream_t st) {
  if (vocab < 1 || !(temp > 0.f)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(sample_row_kernel, dim3(1), dim3(kAcceptThreads), 0, st, logits, vocab, temp, seed, cycle, node, out);
  return hipGetLastError();
}

// ---- commit: greedy acceptance, KV compaction, hand-off -----------------------------------------
// The walk of the greedy acceptance, by one workgroup: every node's argmax (the slices' best, ascending, two threads a row) and the tree into the LDS in one
// trip, then the accepted child of a node is the first one that carries its argmax.  (One wavefront that fetched each node's slices as it came to it
// took 4 us and more, a trip a step.)
struct GreedyWalk { const float *amax_val; const int *amax_idx; int n_slices; const int *tree_tok, *tree_par; int n_nodes; };   // amax_val == nullptr: accepted already
__device__ __forceinline__ void greedy_walk(const GreedyWalk &w, AcceptResult &res) {
  __shared__ int best[kMaxNodes], tok[kMaxNodes], par[kMaxNodes];
  static_assert(kSelThreads == 2 * kMaxNodes, "two threads a row");
  const int t = threadIdx.x, row = t >> 1;
  ValIdx b{-INFINITY, INT_MAX};
  if (row < w.n_nodes)
#pragma unroll 4
    for (int sl = t & 1; sl < w.n_slices; sl += 2) {
      const float x = w.amax_val[(size_t)row * w.n_slices + sl];
      const int c = w.amax_idx[(size_t)row * w.n_slices + sl];
      if (better(x, c, b.v, b.i)) { b.v = x; b.i = c; }
    }
  best_step<1>(b);
  if (row < w.n_nodes) {
    if (t & 1) { tok[row] = w.tree_tok[row]; par[row] = w.tree_par[row]; } else best[row] = b.i;
  }
  __syncthreads();
  if (t < 64) {
    int cur = 0, m = 0;
    if (t == 0) res.node[0] = 0;
    for (int step = 0; step <= kMaxDepth; step++) {
      const int want = best[cur];
      if (t == 0) res.token[m] = want;                       // accepted token, or the bonus when the walk stops
      int child = -1;
      if (m < kMaxDepth)
        for (int c0 = 0; c0 < w.n_nodes && child < 0; c0 += 64) {
          const int c = c0 + t;
          const uint64_t found = __ballot(c > cur && c < w.n_nodes && par[c] == cur && tok[c] == want);
          if (found) child = c0 + __ffsll((unsigned long long)found) - 1;
        }
      if (child < 0) break;
      cur = child; m++;
      if (t == 0) res.node[m] = cur;
    }
    if (t == 0) res.n_acc = m;
  }
}
// One launch: every workgroup walks the tree for itself (or fetches what was accepted), the first n_compact then move the keys and values, the others hand over.
// Three launches of 4 us in a chain before (a cycle of plain decoding has little else that waits for the host).
// Compaction: thread = one 16-byte chunk of one (layer, key|value) row; it moves that chunk for depths 1..m in
// ascending order.  Depth d's destination slot n+d is never a later depth's source (sources
// n+node[d'] have node[d'] > d for d' > d), and a chunk column is owned by one thread, so the
// in-place move is race-free.
// Hand-off: features of root + accepted rows and the matching tokens for the next draft root step.
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
template <typename T>
__global__ __launch_bounds__(kSelThreads) void commit_kernel(GreedyWalk walk, AcceptResult *res, int n_compact, char *kv_base, size_t layer_bytes, size_t kv_bytes, int n_layers,
                                                             int row_bytes, int n, const T *feat, int d, T *pend_feat, int *pend_tok, int *root_tok,
                                                             int *n_committed, AcceptResult *host_res) {
  __shared__ AcceptResult acc;
  constexpr int kWords = sizeof(AcceptResult) / sizeof(int);
  const int t = threadIdx.x;
  if (walk.amax_val != nullptr) greedy_walk(walk, acc);
  else if (t < kWords) ((int *)&acc)[t] = ((const int *)res)[t];
  __syncthreads();
  const int m = acc.n_acc;
  if ((int)blockIdx.x < n_compact) {
    if (m == 0) return;
    const int chunks = row_bytes / 16;
    const size_t total = (size_t)n_layers * 2 * chunks;
    for (size_t w = (size_t)blockIdx.x * kSelThreads + t; w < total; w += (size_t)n_compact * kSelThreads) {
      const int ch = (int)(w % chunks);
      const int kv = (int)((w / chunks) & 1);
      const int l = (int)(w / chunks / 2);
      char *base = kv_base + (size_t)l * layer_bytes + (size_t)kv * kv_bytes + (size_t)ch * 16;
      for (int e = 1; e <= m; e++) {
        const int src = n + acc.node[e], dst = n + e;
        if (src != dst) *(u32x4_t *)(base + (size_t)dst * row_bytes) = *(const u32x4_t *)(base + (size_t)src * row_bytes);
      }
    }
    return;
  }
  const int r = (int)blockIdx.x - n_compact;
  if (r == 0 && t == 0) *n_committed += 1 + m;                // root + accepted tokens are now in the cache
  // the result for the next draft and for the host, straight into its memory: a copy launched behind this kernel was 6 us more to wait for
  if (r == kMaxDepth && t < kWords && (t == 0 || (t - 1) % (kMaxDepth + 1) <= m)) {
    const int x = ((const int *)&acc)[t];
    ((int *)host_res)[t] = x;
    if (walk.amax_val != nullptr) ((int *)res)[t] = x;
  }
  if (r > m) return;
  const T *src = feat + (size_t)acc.node[r] * d;
  T *dst = pend_feat + (size_t)r * d;
  for (int c = t; c < d; c += kSelThreads) dst[c] = src[c];
  if (t == 0) {
    pend_tok[r] = acc.token[r];
    if (r == m) *root_tok = acc.token[m];
  }
}
static hipError_t commit(const GreedyWalk &walk, int dtype, AcceptResult *res, void *kv_base, size_t layer_stride, size_t kv_stride, int n_layers, int row_elems, int n,
                         const void *feat, int d, void *pend_feat, int *pend_tok, int *root_tok, int *n_committed, AcceptResult *host_res, hipStream_t st) {
  const size_t esz = dtype == 1 ? 2 : 4;
  const int row_bytes = (int)(row_elems * esz);
  if (row_bytes % 16 != 0 || n_layers < 1) return hipErrorInvalidValue;
  const size_t total = (size_t)n_layers * 2 * (row_bytes / 16);
  const int blocks = (int)std::min<size_t>(2048, (total + kSelThreads - 1) / kSelThreads);
  const dim3 grid(blocks + kMaxDepth + 1), threads(kSelThreads);
#define SPEC_COMMIT(T) hipLaunchKernelGGL(commit_kernel<T>, grid, threads, 0, st, walk, res, blocks, (char *)kv_base, layer_stride * esz, kv_stride * esz, n_layers, \
                                          row_bytes, n, (const T *)feat, d, (T *)pend_feat, pend_tok, root_tok, n_committed, host_res)
  if (dtype == 1) SPEC_COMMIT(bf16_t); else SPEC_COMMIT(float);
#undef SPEC_COMMIT
  return hipGetLastError();
}
hipError_t launch_commit(int dtype, AcceptResult *res, void *kv_base, size_t layer_stride, size_t kv_stride, int n_layers, int row_elems, int n, const void *feat, int d,
                         void *pend_feat, int *pend_tok, int *root_tok, int *n_committed, AcceptResult *host_res, hipStream_t st) {
  return commit(GreedyWalk{}, dtype, res, kv_base, layer_stride, kv_stride, n_layers, row_elems, n, feat, d, pend_feat, pend_tok, root_tok, n_committed, host_res, st);
}
hipError_t launch_commit_greedy(const float *amax_val, const int *amax_idx, int n_slices, const int *tree_tok, const int *tree_par, int n_nodes, int dtype,
                                AcceptResult *res, void *kv_base, size_t layer_stride, size_t kv_stride, int n_layers, int row_elems, int n, const void *feat, int d,
                                void *pend_feat, int *pend_tok, int *root_tok, int *n_committed, AcceptResult *host_res, hipStream_t st) {
  if (n_nodes < 1 || n_nodes > kMaxNodes || n_slices < 1) return hipErrorInvalidValue;
  return commit(GreedyWalk{amax_val, amax_idx, n_slices, tree_tok, tree_par, n_nodes}, dtype, res, kv_base, layer_stride, kv_stride, n_layers, row_elems, n, feat, d, pend_feat,
                pend_tok, root_tok, n_committed, host_res, st);
}

__global__ __launch_bounds__(kSelThreads) void prefill_handoff_kernel(const u32x4_t *feat, int pieces, const int *root_tok, int n_prompt, u32x4_t *pend_feat,
                                                                      int *pend_tok, int *n_committed, AcceptResult *res, int *host_first) {
  if (threadIdx.x == 0) {
    res->n_acc = 0;
    const int tok = *root_tok;
    *pend_tok = tok; *host_first = tok; *n_committed = n_prompt;
  }
  for (int c = threadIdx.x; c < pieces; c += kSelThreads) pend_feat[c] = feat[c];
}
hipError_t launch_prefill_handoff(const void *feat, int row_bytes, const int *root_tok, int n_prompt, void *pend_feat, int *pend_tok,
                                  int *n_committed, AcceptResult *res, int *host_first, hipStream_t st) {
  if (row_bytes < 16 || row_bytes % 16 || n_prompt < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(prefill_handoff_kernel, dim3(1), dim3(kSelThreads), 0, st, (const u32x4_t *)feat, row_bytes / 16, root_tok, n_prompt,
                     (u32x4_t *)pend_feat, pend_tok, n_committed, res, host_first);
  return hipGetLastError();
}

__global__ __launch_bounds__(64) void pending_rows_kernel(const AcceptResult *res, const int *n_committed, const int *pend_tok, int rows, int *token, int *src,
                                                          int *pos, int *slot, int *depth, int *base) {
  const int i = threadIdx.x;
  if (i >= rows) return;
  const int m = res->n_acc, n = *n_committed, first = n - 1 - m, p = max(m - i, 0);
  token[i] = pend_tok[p]; src[i] = p;
  pos[i] = first + p + 1;
  slot[i] = i <= m ? first + p : n + (i - m - 1);
  depth[i] = p;
  if (i == 0) *base = first;
}
hipError_t launch_pending_rows(const AcceptResult *res, const int *n_committed, const int *pend_tok, int rows, int *token, int *src, int *pos, int *slot,
                               int *depth, int *base, hipStream_t st) {
  if (rows < 1 || rows > kMaxDepth + 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(pending_rows_kernel, dim3(1), dim3(64), 0, st, res, n_committed, pend_tok, rows, token, src, pos, slot, depth, base);
  return hipGetLastError();
}

}  // namespace spec
