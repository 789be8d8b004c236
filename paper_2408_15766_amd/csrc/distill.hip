// Top-K distillation loss (Sec. 3.1, Eq. 1) and the whole-vocabulary cross-entropy, from two fp32 logit
// rows per position: zq (target) and zp (draft), both produced by the LM-head GEMM.
//
//   loss_topk = - sum over the K tokens x of largest zq of  softmax(zq)(x) * log_softmax(zp)(x)
//   loss_ce   = - sum over all tokens                        of the same product
//
// Every logit is read once.  Stage 1, one workgroup per (slice of kTopkSlice tokens, position): the
// slice's softmax statistics of both rows, the cross term sum exp(zq - max) * zp, and the slice's K best
// target logits (as a set) together with the draft logits at the same tokens.  Stage 2, one workgroup per
// position: merges the slices' statistics in ascending order, picks the K best of all candidates and forms both
// losses.  Every sum runs in an order that depends on the data alone.  Ties between equal target logits go to the
// lower token id.
//
// Selection is a search for the K-th largest KEY (value bits in the high word, lower token first in the low word; all
// keys differ), bit by bit from the top with a count of the keys at or above the trial threshold; it ends as soon as the
// count is K.  Ranking candidates against each other costs K rounds or n^2 comparisons instead: 700 positions, vocabulary
// 128256, K = 100: slices 2820 -> 224 us, merge 2385 -> 50 us; 4096 positions, vocabulary 32000, K = 10: 419 -> 322 us
// and 59 -> 69 us.
#include <limits.h>

#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace spec {

namespace {

constexpr int kLossThreads = 256;
constexpr int kLossWaves = kLossThreads / 64;

// The cross terms are summed at this scale: 4096 draft logits at the type's lowest value (a mask) would overflow, and with them slices whose
// weight among the others is 0.
constexpr float kCrossScale = 0x1p-32f;

// scratch per (position, slice): 5 floats of statistics, then K (target logit, token, draft logit) triples
__host__ __device__ inline size_t slice_floats(int k) { return 8 + 3 * (size_t)k; }

// The largest t (from the top bit down) with count(t) >= k, where count(t) = number of keys >= t; stops early at a t with
// exactly k (up to `more` above k).  Keys differ, so exactly k of them are >= the result if there are k keys at all; otherwise
// the result is 0.
template <int LAST = 0, typename Count>                      // LAST: lowest bit looked at
__device__ __forceinline__ uint64_t kth_key(int k, Count count, int more = 0) {
  uint64_t t = 0;
  for (int bit = 63; bit >= LAST; bit--) {
    const uint64_t trial = t | (1ull << bit);
    const int n = count(trial);
    if (n >= k) t = trial;
    if (n >= k && n <= k + more) break;
  }
  return t;
}
template <int N, typename K>
__device__ __forceinline__ int wave_count(const K (&key)[N], K t) {
  int n = 0;
#pragma unroll
  for (int e = 0; e < N; e++) n += __popcll(__ballot(key[e] >= t));
  return n;
}
// ... over the workgroup's WAVES wavefronts; sh: two sets of WAVES ints, alternating (one barrier per count)
template <int WAVES>
__device__ __forceinline__ int block_total(int wave_n, int (*sh)[WAVES], int &turn) {
  if constexpr (WAVES == 1) return wave_n;
  turn ^= 1;
  if ((threadIdx.x & 63) == 0) sh[turn][threadIdx.x >> 6] = wave_n;
  __syncthreads();
  int n = 0;
#pragma unroll
  for (int w = 0; w < WAVES; w++) n += sh[turn][w];
  return __builtin_amdgcn_readfirstlane(n);
}
__device__ __forceinline__ float key_value(uint64_t key) {
  const uint32_t u = (uint32_t)(key >> 32);
  return __uint_as_float(u ^ ((u >> 31) ? 0x80000000u : 0xFFFFFFFFu));
}
__device__ __forceinline__ void put_candidate(float *out, int pos, uint64_t key, float zp) {
  out[8 + 3 * pos + 0] = key ? key_value(key) : -INFINITY;
  out[8 + 3 * pos + 1] = __int_as_float(key ? 0x7FFFFFFF - (int)(uint32_t)key : INT_MAX);
  out[8 + 3 * pos + 2] = key ? zp : 0.f;
}

constexpr int kWaveCand = 128;                               // places for a wavefront's tokens at or above the bound
struct SliceShared {
  float red_max[kLossWaves][2], red_sum[kLossWaves][4];
  __attribute__((aligned(16))) uint32_t tmax[kLossThreads];
  uint64_t ckey[kLossWaves][kWaveCand];
  float czp[kLossWaves][kWaveCand];
  float tau;
  int cnt[2][kLossWaves];
};

// One slice of one position.  EDGE: the slice reaches past the vocabulary (the last one); only there token numbers are tested.
//
// Bound: vector instructions, then the logits' way from the last-level cache (eight 16-byte loads per thread in flight).
// The candidates are found by comparing logits with a bound (one instruction a token; keys are built for those that pass), and
// their places by the masks of these comparisons, most of which are empty; each wavefront lists its own, so one barrier
// stands between finding and choosing.  512 positions, vocabulary 32000, K = 10, between two LM-head products: with a key for every
// token and the places counted over the workgroup first 37.9 us, now 35.8 (the reads and maxima alone 20.6); 188 positions,
// vocabulary 128256, K = 100: 69 -> 54.5.
// The exponentials are expf()'s, two thirds of the vector instructions.  2^(x * log2 e) with one correction takes 30.5 us, but errs by up to
// 3.9 units of the last place where expf() errs by 0.86 (all arguments from -104 to 0), and has no value below 2^-126 nor for
// differences that overflow when scaled; a form as exact as expf(), with one reduction of the argument and no range checks, takes 34.6.
template <bool EDGE>
__device__ __forceinline__ void loss_slice(const float *rq, const float *rp, int ldz, int vocab, int k, int c0, float *out, SliceShared &sh) {
  constexpr int PER = kTopkSlice / kLossThreads;   // 16
  constexpr int C4 = PER / 4;
  typedef __attribute__((ext_vector_type(4))) float f32x4_t;
  static_assert(kLossWaves == 4, "the reductions below combine four wavefronts");
  auto &red_max = sh.red_max;
  auto &red_sum = sh.red_sum;
  auto &tmax = sh.tmax;
  auto &ckey = sh.ckey;
  auto &czp = sh.czp;
  auto &tau_s = sh.tau;
  auto &cnt = sh.cnt;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int t = threadIdx.x;
  // element 4 * i + j of a thread is token c0 + i * 1024 + 4 * t + j; rows are 256-byte aligned and ldz is a multiple of 64
  auto token = [&](int e) { return c0 + (e >> 2) * (4 * kLossThreads) + 4 * t + (e & 3); };
  auto inside = [&](int e) { return !EDGE || token(e) < vocab; };
  float vq[PER], vp[PER];
#pragma unroll
  for (int i = 0; i < C4; i++) {
    const int c = EDGE ? min(token(4 * i), ldz - 4) : token(4 * i);   // past the row: any of its values, masked below
    const f32x4_t q4 = *(const f32x4_t *)(rq + c), p4 = *(const f32x4_t *)(rp + c);
#pragma unroll
    for (int j = 0; j < 4; j++) { vq[4 * i + j] = q4[j]; vp[4 * i + j] = p4[j]; }
  }
#pragma unroll
  for (int e = 0; e < PER; e++)
    if (!inside(e)) vq[e] = vp[e] = -INFINITY;
  // two workgroup-wide reductions, each over several quantities at once (wavefront results in LDS, then every
  // thread combines the four wavefronts in the same fixed order)
  float mq = vq[0], mp = vp[0];
#pragma unroll
  for (int e = 1; e < PER; e++) { mq = fmaxf(mq, vq[e]); mp = fmaxf(mp, vp[e]); }
  // the best key (value word) of each thread: the K-th largest of these 256 bounds the K-th largest logit from below
  tmax[t] = inside(0) ? (uint32_t)(order_key(mq, 0) >> 32) : 0u;
  mq = wave_max(mq);
  mp = wave_max(mp);
  if (lane == 0) { red_max[wave][0] = mq; red_max[wave][1] = mp; }
  __syncthreads();
  mq = fmaxf(fmaxf(red_max[0][0], red_max[1][0]), fmaxf(red_max[2][0], red_max[3][0]));
  mp = fmaxf(fmaxf(red_max[0][1], red_max[1][1]), fmaxf(red_max[2][1], red_max[3][1]));
  if (wave == 0) {
    typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
    const u32x4_t m4 = *(const u32x4_t *)(tmax + 4 * lane);
    const uint32_t m[4] = {m4.x, m4.y, m4.z, m4.w};
    const uint64_t tau = kth_key<32>(k, [&](uint64_t x) { return wave_count(m, (uint32_t)(x >> 32)); }, 8);
    if (lane == 0) tau_s = tau ? key_value(tau) : -INFINITY;  // fewer than k threads with tokens: every token passes
  }
  float sq = 0.f, sp = 0.f, cross = 0.f;
  const float q0 = mq == -INFINITY ? 0.f : mq, p0 = mp == -INFINITY ? 0.f : mp;   // a slice without any probability adds zeros
#pragma unroll
  for (int e = 0; e < PER; e++) {
    const float wq = expf(vq[e] - q0);                       // 0 for padding
    sq += wq;
    sp += expf(vp[e] - p0);
    cross = inside(e) ? fmaf(wq, vp[e], cross) : cross;
  }
  cross = cross * kCrossScale;
  if (__any(!(fabsf(cross) < INFINITY))) {                   // (also a NaN, which stays one)
    cross = 0.f;
#pragma unroll
    for (int e = 0; e < PER; e++) cross = inside(e) ? fmaf(expf(vq[e] - q0) * kCrossScale, vp[e], cross) : cross;
  }
  sq = wave_sum(sq);
  sp = wave_sum(sp);
  cross = wave_sum(cross);
  if (lane == 0) { red_sum[wave][0] = sq; red_sum[wave][1] = sp; red_sum[wave][2] = cross; }
  __syncthreads();
  if (t == 0) {
    out[0] = mq; out[2] = mp;
    out[1] = ((red_sum[0][0] + red_sum[1][0]) + red_sum[2][0]) + red_sum[3][0];
    out[3] = ((red_sum[0][1] + red_sum[1][1]) + red_sum[2][1]) + red_sum[3][1];
    out[4] = ((red_sum[0][2] + red_sum[1][2]) + red_sum[2][2]) + red_sum[3][2];
  }

  // hides from the compiler that these are the values of before: masks and token numbers of all sixteen tokens are
  // then formed where they are used instead of being held in registers
  auto seen = [&] {
#pragma unroll
    for (int e = 0; e < PER; e++) asm volatile("" : "+v"(vq[e]));
    asm volatile("" : "+v"(t), "+s"(vocab));
  };
  // put(position, e) for the wavefront's tokens with pass(e), in a fixed order from `pos` on; the position behind the last
  auto compact = [&](int pos, auto pass, auto put) {
#pragma unroll
    for (int e = 0; e < PER; e++) {
      const uint64_t mask = __ballot(pass(e));
      if (mask) {
        if (pass(e)) put(pos + __popcll(mask & ((1ull << lane) - 1ull)), e);
        pos += __popcll(mask);
      }
    }
    return pos;
  };
  // The tokens at or above the bound: about K, unless large logits sit together in few threads or tie.  NaNs pass.
  const float tau = tau_s;
  seen();
  const int mine = compact(0, [&](int e) { return inside(e) && !(vq[e] < tau); }, [&](int pos, int e) {
    if (pos < kWaveCand) { ckey[wave][pos] = order_key(vq[e], token(e)); czp[wave][pos] = vp[e]; }
  });
  if (lane == 0) cnt[0][wave] = mine;
  __syncthreads();
  const int n0 = cnt[0][0], n1 = cnt[0][1], n2 = cnt[0][2], n3 = cnt[0][3];
  const int n_pass = __builtin_amdgcn_readfirstlane(n0 + n1 + n2 + n3);
  const int n_most = __builtin_amdgcn_readfirstlane(max(max(n0, n1), max(n2, n3)));
  if (n_pass <= 256 && n_most <= kWaveCand) {
    if (wave != 0) return;
    auto finish = [&](auto per) {                             // the K best of up to 64 * per candidates
      constexpr int N = decltype(per)::value;
      uint64_t ck[N];
      float cz[N];
#pragma unroll
      for (int i = 0; i < N; i++) {
        const int c = lane + 64 * i;                          // the wavefronts' tokens one behind the other
        const int w = (c >= n0) + (c >= n0 + n1) + (c >= n0 + n1 + n2);
        const int at = c - (w > 0 ? n0 : 0) - (w > 1 ? n1 : 0) - (w > 2 ? n2 : 0);
        ck[i] = 0ull;
        if (c < n_pass) { ck[i] = ckey[w][at]; cz[i] = czp[w][at]; }
      }
      uint64_t thr = 1;
      if (n_pass > k) thr = kth_key(k, [&](uint64_t x) { return wave_count(ck, x); });
      int pos = 0;
#pragma unroll
      for (int i = 0; i < N; i++) {
        const uint64_t mask = __ballot(ck[i] >= thr);
        if (ck[i] >= thr) put_candidate(out, pos + __popcll(mask & ((1ull << lane) - 1ull)), ck[i], cz[i]);
        pos += __popcll(mask);
      }
      for (int i = pos + lane; i < k; i += 64) put_candidate(out, i, 0ull, 0.f);   // the slice has fewer than k tokens
    };
    if (n_pass <= 64) finish(std::integral_constant<int, 1>{});
    else finish(std::integral_constant<int, 4>{});
    return;
  }
  seen();                                                     // more tokens than k pass: the slice has k tokens
#pragma unroll
  for (int e = 0; e < PER; e++)                               // value words; 0 (below every logit's) past the vocabulary
    vq[e] = __uint_as_float(inside(e) ? (uint32_t)(order_key(vq[e], 0) >> 32) : 0u);
  auto key = [&](int e) { return (uint64_t)__float_as_uint(vq[e]) << 32 | (uint32_t)(0x7FFFFFFF - token(e)); };
  int turn = 0;
  const uint64_t thr = kth_key(k, [&](uint64_t x) {
    int n = 0;
    seen();                                                   // keeps the token numbers of all sixteen out of registers
#pragma unroll
    for (int e = 0; e < PER; e++) n += __popcll(__ballot(key(e) >= x));
    return block_total<kLossWaves>(n, cnt, turn);
  });
  int n = 0, pos = 0;
#pragma unroll
  for (int e = 0; e < PER; e++) n += __popcll(__ballot(key(e) >= thr));
  __syncthreads();
  if (lane == 0) cnt[0][wave] = n;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kLossWaves; w++) pos += w < wave ? cnt[0][w] : 0;
  seen();
  compact(pos, [&](int e) { return key(e) >= thr; }, [&](int at, int e) { put_candidate(out, at, key(e), vp[e]); });
}
__global__ __launch_bounds__(kLossThreads, 7) void loss_slice_kernel(const float *zq, const float *zp, int ldz, int vocab, int k,
                                                                   int n_slices, float *scratch) {
  __shared__ SliceShared sh;
  const int slice = blockIdx.x, rowi = blockIdx.y, c0 = slice * kTopkSlice;
  const float *rq = zq + (size_t)rowi * ldz, *rp = zp + (size_t)rowi * ldz;
  float *out = scratch + ((size_t)rowi * n_slices + slice) * slice_floats(k);
  if (c0 + kTopkSlice <= vocab) loss_slice<false>(rq, rp, ldz, vocab, k, c0, out, sh);
  else loss_slice<true>(rq, rp, ldz, vocab, k, c0, out, sh);
}

constexpr int kLossMaxCand = 4096;
template <int WAVES, int PER>
__global__ __launch_bounds__(WAVES * 64) void loss_merge_kernel(int k, int n_slices, const float *scratch, float *loss_topk, float *loss_ce) {
  __shared__ float sh[4];                                    // lse_q, lse_p, cross / sum_q
  __shared__ float shv[16];
  __shared__ int cnt[2][WAVES];
  const int rowi = blockIdx.x, t = threadIdx.x;
  const float *base = scratch + (size_t)rowi * n_slices * slice_floats(k);
  const int n_cand = n_slices * k;
  auto cand = [&](int id) { return base + (size_t)(id / k) * slice_floats(k) + 8 + 3 * (id % k); };
  uint64_t key[PER];
#pragma unroll
  for (int e = 0; e < PER; e++) {
    const int id = t + e * WAVES * 64;
    key[e] = 0ull;
    if (id < n_cand) { const float *c = cand(id); key[e] = order_key(c[0], __float_as_int(c[1])); }
  }
  if (t < 64) {                                              // slices in ascending groups of 64, fixed butterfly inside
    float mq = -INFINITY, mp = -INFINITY;
    for (int sl = t; sl < n_slices; sl += 64) {
      const float *s = base + (size_t)sl * slice_floats(k);
      mq = fmaxf(mq, s[0]); mp = fmaxf(mp, s[2]);
    }
    mq = wave_max(mq); mp = wave_max(mp);
    float sq = 0.f, sp = 0.f, cr = 0.f;
    for (int s0 = 0; s0 < n_slices; s0 += 64) {
      const int sl = s0 + t;
      const float *s = base + (size_t)sl * slice_floats(k);
      const bool in = sl < n_slices;
      const float fq = in ? expf(s[0] - mq) : 0.f;
      sq += wave_sum(in ? s[1] * fq : 0.f);
      sp += wave_sum(in ? s[3] * expf(s[2] - mp) : 0.f);
      cr += wave_sum(in ? s[4] * fq : 0.f);
    }
    if (t == 0) { sh[0] = mq + logf(sq); sh[1] = mp + logf(sp); sh[2] = cr / sq * (1.f / kCrossScale); }
  }
  int turn = 0;
  const uint64_t thr = kth_key(k, [&](uint64_t x) { return block_total<WAVES>(wave_count(key, x), cnt, turn); });
  __syncthreads();
  const float lse_q = sh[0], lse_p = sh[1];
  float acc = 0.f;
#pragma unroll
  for (int e = 0; e < PER; e++)
    if (key[e] >= thr && key[e] != 0ull) acc += expf(key_value(key[e]) - lse_q) * (cand(t + e * WAVES * 64)[2] - lse_p);
  acc = block_sum(acc, shv);
  if (t == 0) {
    loss_topk[rowi] = -acc;
    loss_ce[rowi] = lse_p - sh[2];                           // - sum q (zp - lse_p)
  }
}

// out[0] = sum of a[0..n), out[1] = sum of b[0..n); one workgroup, fixed order
__global__ __launch_bounds__(kLossThreads) void loss_total_kernel(const float *a, const float *b, int n, float *out) {
  __shared__ float shv[16];
  float sa = 0.f, sb = 0.f;
  for (int i = threadIdx.x; i < n; i += kLossThreads) { sa += a[i]; sb += b[i]; }
  sa = block_sum(sa, shv);
  sb = block_sum(sb, shv);
  if (threadIdx.x == 0) { out[0] = sa; out[1] = sb; }
}

}  // namespace

size_t topk_loss_scratch_floats(int rows, int vocab, int k) {
  const int n_slices = (vocab + kTopkSlice - 1) / kTopkSlice;
  return (size_t)rows * n_slices * slice_floats(k);
}

hipError_t launch_topk_loss_slices(const float *zq, const float *zp, int ldz, int rows, int vocab, int k, float *scratch, hipStream_t st) {
  const int n_slices = (vocab + kTopkSlice - 1) / kTopkSlice;
  if (rows < 1 || rows > 65535 || vocab < 1 || ldz < vocab || ldz % 64 || ((uintptr_t)zq & 15) || ((uintptr_t)zp & 15) || k < 1 || k > kLossMaxK || k > vocab || n_slices * k > kLossMaxCand)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(loss_slice_kernel, dim3(n_slices, rows), dim3(kLossThreads), 0, st, zq, zp, ldz, vocab, k, n_slices, scratch);
  return hipGetLastError();
}

hipError_t launch_topk_loss_merge(int rows, int vocab, int k, const float *scratch, float *loss_topk, float *loss_ce, hipStream_t st) {
  const int n_slices = (vocab + kTopkSlice - 1) / kTopkSlice, n_cand = n_slices * k;
  if (rows < 1 || vocab < 1 || k < 1 || k > kLossMaxK || k > vocab || n_cand > kLossMaxCand) return hipErrorInvalidValue;
  // one wavefront needs no barriers: up to four candidates per lane
  if (n_cand <= 256) hipLaunchKernelGGL((loss_merge_kernel<1, 4>), dim3(rows), dim3(64), 0, st, k, n_slices, scratch, loss_topk, loss_ce);
  else if (n_cand <= 1024) hipLaunchKernelGGL((loss_merge_kernel<4, 4>), dim3(rows), dim3(256), 0, st, k, n_slices, scratch, loss_topk, loss_ce);
  else hipLaunchKernelGGL((loss_merge_kernel<16, 4>), dim3(rows), dim3(1024), 0, st, k, n_slices, scratch, loss_topk, loss_ce);
  return hipGetLastError();
}

hipError_t launch_loss_total(const float *loss_topk, const float *loss_ce, int rows, float *out, hipStream_t st) {
  hipLaunchKernelGGL(loss_total_kernel, dim3(1), dim3(kLossThreads), 0, st, loss_topk, loss_ce, rows, out);
  return hipGetLastError();
}

}  // namespace spec
