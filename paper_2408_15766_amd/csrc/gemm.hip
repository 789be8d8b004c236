// Weight-streaming skinny GEMM for gfx950:  P[s][i][col] = sum_{k in split s} X[i][k] * W[col][k]
//
// Every projection of the decode path (QKV, O, gate/up, down, draft fc, LM head)
// multiplies a handful of token rows (M <= 128 per tile: the verified tree, the draft
// frontier, or one row in plain decoding) by a weight matrix that is read once.
// The step is bound by HBM bandwidth (about 2*M flop per weight byte pair), so
// the design goal is to keep many 16-byte weight loads in flight per lane and
// never touch a weight twice; the matrix cores are used only because M ~ 60
// is too much for the vector ALUs at that rate.
//
// Layout of one MFMA step (v_mfma_f32_32x32x16_bf16; fp32 storage has a kernel of its own, gemm_f32_kernel):
//   A operand = 32 token rows   x k-slice   (from the X slab staged in LDS)
//   B operand = 32 weight rows  x k-slice   (straight from global memory)
//   D         = lane (c = lane%32, g = lane/32) holds weight row c of the
//               wave's 32-row block for tokens 8*(v/4) + 4*g + v%4, v = 0..15
// Weights are read in the library's PACKED layout (pack_weight_kernel below): the
// matrix is cut into tiles of 32 rows x KI k-elements (8 KiB; KI = 128 bf16 / 64 fp32),
// tiles of one 32-row block are consecutive along k, and inside a tile the 16-byte piece
// that lane (c, g) needs for MFMA step j sits at byte j*1024 + lane*16.  One wave-wide
// load instruction therefore reads 1 KiB of consecutive bytes (eight full cache lines),
// and a wave streams one contiguous region from start to end: measured on MI355X this
// is worth ~1.4x in achieved HBM bandwidth over reading the same 16-byte pieces from a
// row-major matrix (64 partial lines per instruction).  Piece (c, g, j) of tile (rb, it)
// holds W[rb*32 + c][it*KI + g*KI/2 + j*EPL .. + EPL), zero beyond the matrix, so neither
// ragged rows nor a ragged K need a special path.  The k indices of one MFMA are not
// contiguous, which is harmless because A and B are indexed by the same (g, element) pair.
//
// Each wave owns one 32-row block of W for the workgroup's K range and all
// token blocks; the four or eight waves of a workgroup share the X slab.  Which blocks a
// workgroup takes is the launch's choice (adjacent ones, or fewer than it has waves, spread so
// that every compute unit has a workgroup: launch_stream).  Weight loads
// run kStages - 1 iterations ahead through a register ring; the X slab is
// double-buffered in LDS and prefetched one slab ahead through registers.
//
// Determinism: the value of P[s][i][col] depends only on row i of X, row col of
// W and the K split, never on M, on the position of the row in its tile or on
// other rows, so a token computes bit-identical results alone (plain decoding)
// or inside a tree.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace spec {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;   // native vector: stays in registers (SSA), unlike HIP's u32x4_t struct

#ifndef SPEC_GEMM_WAVES
#define SPEC_GEMM_WAVES 4
#endif
#ifndef SPEC_GEMM_SLAB_ITERS
#define SPEC_GEMM_SLAB_ITERS 2
#endif
#ifndef SPEC_GEMM_STAGES
#define SPEC_GEMM_STAGES 3
#endif
constexpr int kGemmWaves = SPEC_GEMM_WAVES;         // waves per workgroup
constexpr int kStages = SPEC_GEMM_STAGES;           // register ring: weight loads run kStages - 1 iterations ahead
constexpr int kGemmThreads = kGemmWaves * kWave;
constexpr int kLaneBytes = 128;                     // contiguous weight bytes per lane per iteration
constexpr int kSlabIters = SPEC_GEMM_SLAB_ITERS;    // iterations per LDS slab
constexpr int kSlabRowBytes = 2 * kLaneBytes * kSlabIters;   // 512 B of k per token row per slab
constexpr int kSlabStride = kSlabRowBytes + 16;     // +16 B: conflict-free 16-byte LDS reads
constexpr int kTileBytes = 32 * 2 * kLaneBytes;     // one packed tile: 32 rows x 256 B of k

template <typename T> struct GemmTraits;
template <> struct GemmTraits<bf16_t> { static constexpr int kEpl = 8; };   // elements per 16 bytes
template <> struct GemmTraits<float>  { static constexpr int kEpl = 4; };

__device__ __forceinline__ void mfma_step(f32x16_t &acc, const u32x4_t &x, const u32x4_t &w, bf16_t) {
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, x), __builtin_bit_cast(bf16x8_t, w), acc, 0, 0, 0);
}

constexpr int gcd_ce(int a, int b) { return b == 0 ? a : gcd_ce(b, a % b); }
template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F &&f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// SwiGLU epilogue of a block of the gate/up matrix.  Lane c < 16 holds the gate sums of column col = block * 16 + c
// and lane c + 16 the up sums of the same column and tokens.  Each finishes half of the values (the low lane the
// accumulator entries v < 8, the high lane v >= 8): swapping the odd rows of 16 lanes of entry v with the even ones of entry 8 + v
// leaves the gate sum in one register and the up sum in the other, in both.  Then lanes of adjacent columns swap one of two token rows
// and write two columns as one word, 32 bits per lane of every store.  All on the vector unit: through the LDS crossbar (two
// round trips a value, half the lanes idle in the stores) it was 2 to 3 us of a launch: 7B gate/up of 60 rows 34.1 -> 33.1 us,
// ten rows 30.1 -> 28.9, 8B 42.8 -> 41.1 and 40.4 -> 38.7, 13B 50.9 -> 49.5 and 45.2 -> 44.0.
// act: the block's first token row, column col (even ones 4-byte aligned where f is even).
template <int TB>
__device__ __forceinline__ void swiglu_epilogue(const f32x16_t (&acc)[TB], bf16_t *act, int f, int col, bool store, int m_loc, int c, int g) {
  const bool odd = c & 1;
  const int v0 = c >= 16 ? 8 : 0;
  const bool pairs = (f & 1) == 0;                            // (then a column and its neighbour exist both or neither)
  uint32_t *const words = (uint32_t *)(act - (odd ? 1 : 0));
#pragma unroll
  for (int t = 0; t < TB; t++) {
    float r[8];
#pragma unroll
    for (int v8 = 0; v8 < 8; v8++) {
      const auto w = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[t][v8]), __float_as_uint(acc[t][8 + v8]), false, false);
      r[v8] = silu_mul(__uint_as_float(w[0]), __uint_as_float(w[1]));
    }
#pragma unroll
    for (int q = 0; q < 4; q++) {                             // entries v0 + 2 q (kept by the even lane) and v0 + 2 q + 1
      const int v = v0 + 2 * q, i = t * 32 + 8 * (v >> 2) + 4 * g + (v & 3);
      if (pairs) {
        const float mine = odd ? r[2 * q + 1] : r[2 * q], got = dpp_f32<0xB1>(odd ? r[2 * q] : r[2 * q + 1]);   // quad_perm [1,0,3,2]
        const int row = i + (odd ? 1 : 0);
        if (store && row < m_loc) store_through(words + (uint32_t)row * (uint32_t)f / 2u, pack_bf16x2(odd ? got : mine, odd ? mine : got));
      } else {
        if (store && i < m_loc) act[(size_t)i * f].v = f32_to_bf16_bits(r[2 * q]);
        if (store && i + 1 < m_loc) act[(size_t)(i + 1) * f].v = f32_to_bf16_bits(r[2 * q + 1]);
      }
    }
  }
}

// First slab of split y, floor(y * slabs / n_split).  With slabs = slab_base * n_split + slab_rem that is y * slab_base + floor(y * slab_rem /
// n_split), and the quotient is the high word of a product with ceil(2^64 / n_split): exact, since the product of dividend and divisor
// stays below 2^64 (n_split = 1: slab_rem = 0; n_split is a grid dimension, up to 65535).  A 64-bit division is some 150 instructions, and two of them stood ahead of a launch's
// first load.
__device__ __forceinline__ int slab_begin(const GemmArgs &a, int y) {
  const uint32_t x = (uint32_t)y * (uint32_t)a.slab_rem;
  return y * a.slab_base + (int)(((uint64_t)x * a.split_hi + __umulhi(x, a.split_lo)) >> 32);
}

// PAIR: a second set of m rows (x2 -> part2) follows the first as rows m .. 2m-1 of the token tile.
template <typename T, int TB, bool PAIR, int WAVES>
__global__ __launch_bounds__(WAVES * kWave, WAVES > 4 ? WAVES / 4 : (TB <= 2 && kStages <= 3) ? 2 : 1) void gemm_stream_kernel(GemmArgs a) {
  constexpr int kThreads = WAVES * kWave;
  constexpr int EPL = GemmTraits<T>::kEpl;
  constexpr int KI = 2 * kLaneBytes / (int)sizeof(T);         // k elements per iteration
  constexpr int XCH = TB * 32 * (kSlabRowBytes / 16) / kThreads;   // 16-byte X chunks per thread per slab
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  constexpr int kSlabBytes = TB * 32 * kSlabStride;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = lane & 31, g = lane >> 5;

  // which 32-row block of which weight segment this wave streams (no dynamic indexing of the
  // argument struct: that would push it to private memory).
  // A wave past the last block recomputes the last block and stores nothing, so that every wave
  // runs the same branch-free loop and the same barriers.
  // SwiGLU mode streams the one gate/up matrix (see pack_gate_up_kernel): a block holds 16 gate rows in the lanes
  // c < 16 and the up rows of the same 16 columns in the lanes c >= 16; seg_rows[0] is the number of columns.
  const int bx = blockIdx.x, by = blockIdx.y;
  const int m_loc = PAIR ? 2 * a.m : a.m;                      // (more than 128 rows: gemm_mm_kernel)
  const bool swiglu = a.act != nullptr;
  const int e0 = a.seg_blocks[0], e1 = e0 + (a.nseg > 1 ? a.seg_blocks[1] : 0);
  const int blk_raw = bx * a.blk_per_wg + wave * a.blk_per_wave;   // adjacent blocks, or strided over more workgroups: see launch_stream
  const bool active = blk_raw < a.total_blocks;
  const int blk = active ? blk_raw : a.total_blocks - 1;
  const int seg = blk < e0 ? 0 : (blk < e1 ? 1 : 2);
  const int b0 = seg == 0 ? 0 : (seg == 1 ? e0 : e1);
  const int seg_rows = seg == 0 ? a.seg_rows[0] : (seg == 1 ? a.seg_rows[1] : a.seg_rows[2]);
  const int seg_col0 = seg == 0 ? a.seg_col0[0] : (seg == 1 ? a.seg_col0[1] : a.seg_col0[2]);
  const void *seg_w = seg == 0 ? a.seg_w[0] : (seg == 1 ? a.seg_w[1] : a.seg_w[2]);
  const int row = (blk - b0) * 32 + c;

  // K splits are balanced to within one slab: split y covers slabs [y*S/n, (y+1)*S/n)
  const int n_it_total = (a.in + KI - 1) / KI;                         // tiles along k (K zero-padded to KI)
  const int it_begin = slab_begin(a, by) * kSlabIters;
  const int it_end = min(n_it_total, slab_begin(a, by + 1) * kSlabIters);
  const int k_begin = it_begin * KI;
  const int n_iter = it_end - it_begin;
  const int n_slab = (n_iter + kSlabIters - 1) / kSlabIters;
  // A wave without a block of its own only helps to stage the X slabs (same barriers, no weight loads, no MFMAs).
  const int n_iter_w = __builtin_amdgcn_readfirstlane(active ? n_iter : 0);
  // this wave's stream: tiles it_begin .. it_end of row block (blk - b0), one contiguous region
  const char *wstream = (const char *)seg_w + ((size_t)(blk - b0) * n_it_total + it_begin) * (size_t)kTileBytes + lane * 16;

  f32x16_t acc[TB];
#pragma unroll
  for (int t = 0; t < TB; t++)
#pragma unroll
    for (int v = 0; v < 16; v++) acc[t][v] = 0.f;

  u32x4_t ring[kStages][8];
  u32x4_t xr[XCH];

  // Every tile is complete in the packed layout (zero-padded), so weight loads need no guard and
  // nothing forces a wait between a load and its use two iterations later.  X never needs
  // zeroing either: out-of-range X addresses are clamped to valid finite data that meets a zero
  // weight or a token row that is never stored.
  auto load_w = [&](u32x4_t (&dst)[8], int it) __attribute__((always_inline)) {
    const char *p = wstream + (size_t)it * kTileBytes;
#pragma unroll
    for (int j = 0; j < 8; j++) dst[j] = __builtin_nontemporal_load((const u32x4_t *)(p + j * 1024));   // read once: do not keep in cache
  };
  auto load_x = [&](int slab) __attribute__((always_inline)) {
    const int k0 = k_begin + slab * kSlabIters * KI;
#pragma unroll
    for (int i = 0; i < XCH; i++) {
      const int q = tid + i * kThreads;
      const int r = q / (kSlabRowBytes / 16), cc = q % (kSlabRowBytes / 16);
      const int kk = k0 + cc * EPL;
      const bool second = PAIR && r >= a.m && r < m_loc;
      const char *xbase = (const char *)(second ? a.x2 : a.x);
      xr[i] = *(const u32x4_t *)(xbase + ((size_t)(r < m_loc ? (second ? r - a.m : r) : 0) * a.ldx + (kk < a.in ? kk : 0)) * sizeof(T));
    }
  };
  auto store_x = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < XCH; i++) {
      const int q = tid + i * kThreads;
      const int r = q / (kSlabRowBytes / 16), cc = q % (kSlabRowBytes / 16);
      *(u32x4_t *)(lds + buf * kSlabBytes + r * kSlabStride + cc * 16) = xr[i];
    }
  };
  auto compute = [&](const u32x4_t (&w)[8], int buf, int ii) __attribute__((always_inline)) {
    const unsigned char *base = lds + buf * kSlabBytes + c * kSlabStride + ii * (2 * kLaneBytes) + g * kLaneBytes;
#pragma unroll
    for (int j = 0; j < 8; j++) {
#pragma unroll
      for (int t = 0; t < TB; t++) {
        const u32x4_t xf = *(const u32x4_t *)(base + t * 32 * kSlabStride + j * 16);
        mfma_step(acc[t], xf, w[j], T{});
      }
    }
  };

  load_x(0);
#pragma unroll
  for (int it = 0; it < kStages - 1; it++)
    if (it < n_iter_w) load_w(ring[it], it);
  store_x(0);
  __syncthreads();

  // The ring stage of iteration `it` is it % kStages.  A slab is kSlabIters iterations, so kPeriod slabs
  // form one period of the stage pattern and are unrolled with compile-time stage indices
  // (P = slab index mod kPeriod).  Steady state (FAST): every load of the slab is a full, in-range
  // iteration and a next slab exists, so the body has no branch and the compiler keeps exact
  // outstanding-load counts; the last slabs of a stream take the guarded form.
  auto slab = [&](auto p_tag, auto fast_tag, int S) __attribute__((always_inline)) {
    constexpr int P = decltype(p_tag)::value;
    constexpr bool FAST = decltype(fast_tag)::value;
    if (!FAST && S >= n_slab) return;
    const int buf = S & 1;
    const bool more = FAST || S + 1 < n_slab;
    if (more) load_x(S + 1);
#pragma unroll
    for (int ii = 0; ii < kSlabIters; ii++) {
      constexpr int base_stage = (kSlabIters * P) % kStages;
      const int it = S * kSlabIters + ii;
      // stage indices are compile-time after unrolling
      const int st_use = (base_stage + ii) % kStages, st_load = (base_stage + ii + kStages - 1) % kStages;
      if (FAST || it + kStages - 1 < n_iter_w) load_w(ring[st_load], it + kStages - 1);
      __builtin_amdgcn_sched_barrier(0);                     // keep the prefetch ahead of the MFMAs
      if (FAST || it < n_iter_w) compute(ring[st_use], buf, ii);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (more) {
      store_x(buf ^ 1);
      __syncthreads();
    }
  };
  constexpr int kPeriod = kStages / gcd_ce(kStages, kSlabIters), kTail = (kStages + kSlabIters - 2) / kSlabIters + 1;
  auto period = [&](auto fast_tag, int S0) __attribute__((always_inline)) {
    static_for<kPeriod>([&](auto p_tag) __attribute__((always_inline)) { slab(p_tag, fast_tag, S0 + decltype(p_tag)::value); });
  };
  // slabs S whose last prefetch, iteration S*kSlabIters + kSlabIters - 1 + kStages - 1, is in range: all but the last one or two
  const int n_steady = n_iter_w >= kSlabIters + kStages - 1 ? (n_iter_w - kStages + 1) / kSlabIters : 0;
  int s = 0;
  for (; s + kPeriod <= n_steady; s += kPeriod) period(std::true_type{}, s);
  if constexpr (TB <= (PAIR ? 1 : 2)) {
    // The steady slabs left over run FAST too: in the guarded form the waits count on the loads that a branch may have left out, so
    // a slab there waits for what it has just requested, up to three times a stream.  7B down of 60 rows 20.2 -> 19.3 us, of ten 17.2 -> 16.1, 8B down 25.6 ->
    // 24.1, 13B O 14.3 -> 13.9, 7B QKV of ten rows 18.6 -> 18.0.  (More rows leave too few registers: 100 rows -8 to +4 %, pairs of sets spill, 60 positions of a loss 219 -> 251.)
    if (n_iter_w == 0)                                        // no block: only help to stage
      for (int S = 0; S + 1 < n_slab; S++) {
        load_x(S + 1);
        store_x((S & 1) ^ 1);
        __syncthreads();
      }
    else
      static_for<kPeriod>([&](auto r_tag) __attribute__((always_inline)) {   // R steady slabs are left
        constexpr int R = decltype(r_tag)::value;
        if (n_steady - s != R) return;
        static_for<R>([&](auto p_tag) __attribute__((always_inline)) { slab(p_tag, std::true_type{}, s + decltype(p_tag)::value); });
        static_for<kTail>([&](auto t_tag) __attribute__((always_inline)) {
          constexpr int Q = R + decltype(t_tag)::value;
          slab(std::integral_constant<int, Q % kPeriod>{}, std::false_type{}, s + Q);
        });
        s = n_slab + kPeriod;                                 // done: matches no other R
      });
  } else {
    for (; s < n_slab; s += kPeriod) period(std::false_type{}, s);
  }

  if (swiglu) {
    const int col = blk * 16 + (c & 15);
    swiglu_epilogue<TB>(acc, (bf16_t *)a.act + col, seg_rows, col, active && col < seg_rows, m_loc, c, g);
    return;
  }
  if (!active || row >= seg_rows) return;
  const size_t o0 = (size_t)by * a.m_pad * a.ldp + seg_col0 + row;
#pragma unroll
  for (int t = 0; t < TB; t++)
#pragma unroll
    for (int v = 0; v < 16; v++) {
      const int i = t * 32 + 8 * (v >> 2) + 4 * g + (v & 3);
      const bool second = PAIR && i >= a.m;
      if (i < m_loc) store_through(&(second ? a.part2 : a.part)[o0 + (size_t)(second ? i - a.m : i) * a.ldp], acc[t][v]);
    }
}

// ---- one row, bf16 (plain decoding) ---------------------------------------------------------------------
// A row fits the LDS whole (the launch's K range of it), so the wavefronts stream their weights without a barrier, and a launch can make its x by itself:
// every workgroup for itself, while its first weights are on their way.  What a row is made of (the partial sums of the projection before and the residual,
// or the attention's parts) is 20 to 80 KB, read from the caches by all workgroups; as launches of their own the row kernels were 4.7 us each of 92 a layer,
// most of it the way from launch to launch.  (Rows made by one workgroup and handed to the others inside a launch cost more than the launch: 9 us.)
// Sums, norm and merge are the row kernels' operations in their order, and the products run in gemm_stream_kernel's order: same bits.
// Measured (7B shape, us, row kernel and streaming launch / this): O 4.7 + 7.9 / 8.5, gate/up 4.75 + 28.9 / 30.4, QKV 4.75 + 18.0 / 19.8, LM head 4.75 + 41.6 / 42.3;
// plain decoding of 16 tokens behind a prompt of 77 49.4 -> 47.0 ms.  Eight wavefronts share the sums (with four, 256 registers spill: 36 us the gate/up launch; with sixteen
// 37).  More rows do not pay: verify of two 820 -> 814 us (8 layers; 13B, 6 layers 851 -> 883), of four 828 -> 906.
struct NoHead {};
template <int KIND> using HeadArg = std::conditional_t<KIND == kHeadNone, NoHead, GemmHead>;
constexpr int kRowMaxCols = 2 * 4 * kNormThreads;             // widest row of kHeadSums
constexpr int kRowLds = 64 * 1024 - 256;                      // bytes of the row's K range (what a launch may ask for without more ado)
__host__ __device__ inline int row_bytes(int slab_base, int slab_rem) { return (slab_base + (slab_rem ? 1 : 0)) * kSlabRowBytes; }

// The row of launch_reduce_add_norm by THREADS threads: pass q is virtual thread q * THREADS + tid
template <int THREADS>
struct SumsRow {
  static constexpr int kPass = kNormThreads / THREADS, E = kRowMaxCols / (4 * kNormThreads), NS = 4;   // NS: split sums requested at once
  f32x4_t p[E][kPass][NS], res[E][kPass];
  static __device__ __forceinline__ int col(int e, int q) { return (e * kNormThreads + q * THREADS + (int)threadIdx.x) * 4; }
  __device__ __forceinline__ void load(const GemmHead &h) {
#pragma unroll
    for (int e = 0; e < E; e++) {
      if (e * 4 * kNormThreads >= h.d) continue;              // (the same for all)
#pragma unroll
      for (int q = 0; q < kPass; q++) {
        const int c = col(e, q) < h.d ? col(e, q) : 0;
        res[e][q] = *(const f32x4_t *)(h.h_in + c);
#pragma unroll
        for (int s = 0; s < NS; s++) p[e][q][s] = *(const f32x4_t *)(h.part + (size_t)(s < h.n_split ? s : 0) * h.m_pad * h.ldp + c);
      }
    }
  }
  // The normed row's columns [k0, k1) to xl (LDS) and, with `store`, the whole row to x and h_out.  sh: kNormThreads / 64 floats
  __device__ __forceinline__ void finish(const GemmHead &h, unsigned char *xl, int k0, int k1, bf16_t *x, bool store, float *sh) {
    const bf16_t *norm_w = (const bf16_t *)h.norm_w;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    f32x4_t v[E][kPass], nw[E][kPass];
    float ss[kPass] = {};
#pragma unroll
    for (int e = 0; e < E; e++) {
      if (e * 4 * kNormThreads >= h.d) continue;
#pragma unroll
      for (int q = 0; q < kPass; q++) nw[e][q] = (norm_w != nullptr && col(e, q) < h.d) ? load4<bf16_t>(norm_w + col(e, q)) : f32x4_t{1.f, 1.f, 1.f, 1.f};
#pragma unroll
      for (int q = 0; q < kPass; q++) {
        const int c = col(e, q) < h.d ? col(e, q) : 0;
        f32x4_t acc = p[e][q][0];
#pragma unroll
        for (int s = 1; s < NS; s++)
          if (s < h.n_split) acc += p[e][q][s];
        for (int s = NS; s < h.n_split; s++) acc += *(const f32x4_t *)(h.part + (size_t)s * h.m_pad * h.ldp + c);
        v[e][q] = h.residual ? res[e][q] + acc : acc;
        if (col(e, q) < h.d) ss[q] = add_squares(ss[q], v[e][q]);
      }
    }
    float r = 1.f;
    if (norm_w != nullptr) {
#pragma unroll
      for (int q = 0; q < kPass; q++) {
        const float w = wave_sum(ss[q]);
        if (lane == 0) sh[q * (THREADS / kWave) + wave] = w;
      }
      __syncthreads();
      float t = 0.f;
      for (int w = 0; w < kNormThreads / kWave; w++) t += sh[w];
      r = norm_scale(t, h.d, h.eps);
    }
#pragma unroll
    for (int e = 0; e < E; e++)
#pragma unroll
      for (int q = 0; q < kPass; q++) {
        const int c = col(e, q);
        if (c >= h.d) continue;
        f32x4_t o = v[e][q];
        if (norm_w != nullptr) o = o * r * nw[e][q];
        const uint2 u = {pack_bf16x2(o.x, o.y), pack_bf16x2(o.z, o.w)};
        if (c >= k0 && c < k1) *(uint2 *)(xl + (c - k0) * 2) = u;
        if (store) {
          *(f32x4_t *)(h.h_out + c) = v[e][q];
          *(uint2 *)(x + c) = u;
        }
      }
  }
};

// Dynamic LDS: row_bytes(), the row's K range
template <int KIND, int WAVES>
__global__ __launch_bounds__(WAVES * kWave, WAVES > 4 ? WAVES / 4 : 2) void gemm_row_kernel(GemmArgs a, GemmHead head) {
  constexpr int kThreads = WAVES * kWave, KI = 2 * kLaneBytes / (int)sizeof(bf16_t);
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  __shared__ float sh[kNormThreads / kWave];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, c = lane & 31, g = lane >> 5;
  // blocks, segments and K ranges as in gemm_stream_kernel
  const int bx = blockIdx.x, by = blockIdx.y;
  const int e0 = a.seg_blocks[0], e1 = e0 + (a.nseg > 1 ? a.seg_blocks[1] : 0);
  const int blk_raw = bx * a.blk_per_wg + wave * a.blk_per_wave;
  const bool active = blk_raw < a.total_blocks;
  const int blk = active ? blk_raw : a.total_blocks - 1;
  const int seg = blk < e0 ? 0 : (blk < e1 ? 1 : 2);
  const int b0 = seg == 0 ? 0 : (seg == 1 ? e0 : e1);
  const int seg_rows = seg == 0 ? a.seg_rows[0] : (seg == 1 ? a.seg_rows[1] : a.seg_rows[2]);
  const int seg_col0 = seg == 0 ? a.seg_col0[0] : (seg == 1 ? a.seg_col0[1] : a.seg_col0[2]);
  const void *seg_w = seg == 0 ? a.seg_w[0] : (seg == 1 ? a.seg_w[1] : a.seg_w[2]);
  const int row = (blk - b0) * 32 + c;
  const int n_it_total = (a.in + KI - 1) / KI;
  const int it_begin = slab_begin(a, by) * kSlabIters, it_end = min(n_it_total, slab_begin(a, by + 1) * kSlabIters);
  const int n_iter = __builtin_amdgcn_readfirstlane(active ? it_end - it_begin : 0);   // of this wavefront
  const int k0 = it_begin * KI, k1 = min(it_end * KI, a.in);
  const char *wstream = (const char *)seg_w + ((size_t)(blk - b0) * n_it_total + it_begin) * (size_t)kTileBytes + lane * 16;
  u32x4_t ring[kStages][8];
  auto load_w = [&](u32x4_t (&dst)[8], int it) __attribute__((always_inline)) {
    const char *p = wstream + (size_t)it * kTileBytes;
#pragma unroll
    for (int j = 0; j < 8; j++) dst[j] = __builtin_nontemporal_load((const u32x4_t *)(p + j * 1024));
  };
  auto first_weights = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int it = 0; it < kStages - 1; it++)
      if (it < n_iter) load_w(ring[it], it);
  };

  for (int q = k1 + tid; q < it_end * KI; q += kThreads) *(uint16_t *)(lds + (q - k0) * 2) = 0;   // past K: meets zero weights, has to be finite
  if constexpr (KIND == kHeadSums) {
    SumsRow<kThreads> r;
    r.load(head);
    first_weights();
    r.finish(head, lds, k0, k1, (bf16_t *)a.x, bx == 0 && by == 0, sh);
  } else {
    // four columns a thread (of one head: hd is a multiple of 4), all their parts in flight
    const AttnMerge &mg = head.merge;
    const int n_front = attn_parts_covering(bulk_end((mg.base_ptr ? *mg.base_ptr : mg.base) + mg.depth[0])), n_parts = n_front + 1;
    auto columns = [&](int col, auto between) __attribute__((always_inline)) {
      const int at = min(col, a.in - 4), dim = at % mg.hd;
      const float *src = mg.part + (size_t)(at / mg.hd) * mg.max_parts * (mg.hd + 2);
      float2 ml[kHeadMaxParts], lo[kHeadMaxParts], hi[kHeadMaxParts];
#pragma unroll
      for (int t = 0; t < kHeadMaxParts; t++) {
        const float *sp = src + (size_t)(t < n_front ? t : mg.max_parts - 1) * (mg.hd + 2);
        if (t < n_parts) { ml[t] = *(const float2 *)sp; lo[t] = *(const float2 *)(sp + 2 + dim); hi[t] = *(const float2 *)(sp + 4 + dim); }
      }
      between();
      if (col >= k1) return;
      RowMerge rm;
      f32x4_t o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < kHeadMaxParts; t++)
        if (t < n_parts) {
          float w;
          const float turn = rm.step(ml[t].x, ml[t].y, w);
          o.x = fmaf(lo[t].x, w, o.x * turn); o.y = fmaf(lo[t].y, w, o.y * turn);
          o.z = fmaf(hi[t].x, w, o.z * turn); o.w = fmaf(hi[t].y, w, o.w * turn);
        }
      *(uint2 *)(lds + (col - k0) * 2) = uint2{pack_bf16x2(o.x / rm.l, o.y / rm.l), pack_bf16x2(o.z / rm.l, o.w / rm.l)};
    };
    columns(k0 + tid * 4, first_weights);
    for (int col = k0 + (tid + kThreads) * 4; col < k1; col += kThreads * 4) columns(col, []() {});
  }
  __syncthreads();

  f32x16_t acc[1];
#pragma unroll
  for (int v = 0; v < 16; v++) acc[0][v] = 0.f;
  const unsigned char *xl = lds + g * kLaneBytes;             // (all 32 token rows of the products are the one row)
  auto compute = [&](const u32x4_t (&w)[8], int it) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 8; j++) mfma_step(acc[0], *(const u32x4_t *)(xl + it * (2 * kLaneBytes) + j * 16), w[j], bf16_t{});
  };
  int it = 0;
  for (; it + 2 * kStages - 1 <= n_iter; it += kStages)       // every load is in range: no branch, exact waits
#pragma unroll
    for (int u = 0; u < kStages; u++) {
      load_w(ring[(u + kStages - 1) % kStages], it + u + kStages - 1);
      __builtin_amdgcn_sched_barrier(0);
      compute(ring[u], it + u);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
  for (int u = 0; u < 2 * kStages - 2; u++)
    if (it + u < n_iter) {
      if (it + u + kStages - 1 < n_iter) load_w(ring[(u + kStages - 1) % kStages], it + u + kStages - 1);
      compute(ring[u % kStages], it + u);
    }

  if (a.act != nullptr) {
    const int col = blk * 16 + (c & 15);
    swiglu_epilogue<1>(acc, (bf16_t *)a.act + col, seg_rows, col, active && col < seg_rows, 1, c, g);
    return;
  }
  if (active && row < seg_rows && g == 0) store_through(&a.part[(size_t)by * a.m_pad * a.ldp + seg_col0 + row], acc[0][0]);
}

// ---- more than 128 token rows, bf16 (prefill, LM head of the loss) ------------------------------
// Here the matrix cores are the limit, and what holds them up is the arrival of operands.  A workgroup of eight wavefronts
// (two per SIMD, so that one's products cover the other's waits) owns TW*TB 32-token blocks x (8/TW)*WB 32-row weight blocks
// for one K split; a wavefront owns TB x WB of them.  Both operands are copied straight into the LDS, 64 k at a time (half a
// packed tile): X two stages deep (it sits in L2), the weights three (their first touch comes from HBM: two stages are about
// 2 us of cover).  One barrier per stage, placed before the stage's last step: by then every fragment of the stage is in
// registers, so the copies of later stages may overwrite it, and the next stage's first fragments are read while the last
// step's products run.  Each stage buffer is an array of its own: the compiler then knows which copies a read depends on and
// adds no waits to the two written below.  The sums of a row run in the order of gemm_stream_kernel's (k ascending in
// one accumulator).
// Measured (MI355X, us; before = 128 x 256 tiles with the weights streamed through registers): 512 x 12288 x 4096 with 2 splits
// 86 -> 49, 512 x 32000 x 4096 161 -> 119, 4096 x 28672 x 4096 1113 -> 789, 4096 x 4096 x 14336 492 -> 363.
// What limits it (LM head of 2 x 512 rows, 240 us when this was taken; with parts of the loop left out): without the copies into the LDS 194,
// without the fragment reads as well 158, without the barrier no change.  So it is the traffic through the LDS, and the power: the clock falls
// to 1.8 GHz in the large launches, the matrix cores are busy 59 % of the cycles, and products from registers alone run at 1.59 PFLOP/s on
// normally distributed data (2.39 on zeros).  Four wavefronts of 128 x 128 read a third less from the LDS, but one wavefront per SIMD
// pays more at the ends of a tile: the same time at K = 8192, 3 % slower at 4096.
template <int TW, int TB, int WB>
struct MmTile {
  static constexpr int kTok = TW * TB * 32;                   // tokens per workgroup
  static constexpr int kBlocks = 8 / TW * WB;                 // 32-row weight blocks per workgroup
  static constexpr int kX = kTok * 128, kW = kBlocks * 4096;  // bytes of one stage
  static constexpr int kXLoads = kX / 8192, kWLoads = kW / 8192;   // 1 KB copies per wave and stage
};
constexpr int kMmThreads = 512;

// The token tiles of gemm_mm_mixed_kernel, per weight tile and K range: full ones of 256 rows (the last may have fewer, but more than 128), and
// one ragged end of up to 128 rows per set.
struct MmLists { int weight_tiles, set_full, full, ragged; };
__host__ __device__ inline MmLists mm_lists(int m, int sets, int weight_tiles) {
  const int f = m / 256 + (m % 256 > 128 ? 1 : 0);
  return MmLists{weight_tiles, f, sets * f, m % 256 != 0 && m % 256 <= 128 ? sets : 0};
}

typedef __attribute__((address_space(3))) void lds_void;
// 16 bytes per lane from base + voff (lane) + soff (wave-uniform) straight into the LDS, to dst + 16 * lane; dst is wave-uniform
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *base) {
  return __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, 0x7FFFFFFF, 0x00027000);
}
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t base, int voff, int soff, void *dst) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(base, (lds_void *)dst, 16, voff, soff, 0, 0);
}

// Workgroup barrier that waits for nothing else (__syncthreads would also wait for every copy into the LDS under way)
__device__ __forceinline__ void wg_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// A field of the launch's arguments as a value of its own: a choice between two fields must not become a choice between their addresses (that
// would put the arguments into private memory).
template <typename V> __device__ __forceinline__ V pinned(V v) { asm("" : "+s"(v)); return v; }

// FOLD: the workgroup walks all K ranges of its tile one after the other (the copies run on across the borders) and adds up
// the ranges' sums in registers, ((range 0 + range 1) + range 2) + .., the order in which the row kernels add partial sums: the
// bits of n_split sets of partial sums with one set in memory.  The 256 x 256 tile leaves no registers for a second set of sums; 256 x 192 just does.
//
// One tile: token rows from m0 on of the first or second set of rows, weight blocks from bx * kBlocks on, K range by.  xs, ws: the stage buffers.
template <int TW, int TB, int WB, bool FOLD>
__device__ __forceinline__ void mm_tile_body(const GemmArgs &a, int bx, int by, bool second, int m0, unsigned char *xs0, unsigned char *xs1, unsigned char *ws0,
                                             unsigned char *ws1, unsigned char *ws2) {
  using L = MmTile<TW, TB, WB>;
  constexpr int XI = L::kXLoads, WI = L::kWLoads;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 31, g = lane >> 5;
  bx = __builtin_amdgcn_readfirstlane(bx); by = __builtin_amdgcn_readfirstlane(by); m0 = __builtin_amdgcn_readfirstlane(m0);   // scalars, whatever divisions they come from
  const int m_loc = min(a.m - m0, L::kTok);
  const void *const w_0 = pinned(a.seg_w[0]), *const w_1 = pinned(a.seg_w[1]), *const w_2 = pinned(a.seg_w[2]);
  const int rows_0 = pinned(a.seg_rows[0]), rows_1 = pinned(a.seg_rows[1]), rows_2 = pinned(a.seg_rows[2]);
  const int col_0 = pinned(a.seg_col0[0]), col_1 = pinned(a.seg_col0[1]), col_2 = pinned(a.seg_col0[2]);
  const void *const x_0 = pinned(a.x), *const x_1 = pinned(a.x2);
  float *const out_0 = pinned(a.part), *const out_1 = pinned(a.part2);

  const bool swiglu = a.act != nullptr;
  const int e0 = a.seg_blocks[0], e1 = e0 + (a.nseg > 1 ? a.seg_blocks[1] : 0);
  const int n_it_total = (a.in + 127) / 128;
  auto range_begin = [&](int r) { return min(n_it_total, slab_begin(a, r) * kSlabIters); };
  const int it_begin = range_begin(by), it_end = FOLD ? n_it_total : range_begin(by + 1);
  const int n_stage = 2 * (it_end - it_begin);

  auto block_seg = [&](int blk, int &b0) { const int s = blk < e0 ? 0 : (blk < e1 ? 1 : 2); b0 = s == 0 ? 0 : (s == 1 ? e0 : e1); return s; };
  // the 1 KB pieces of the weight blocks that this wave copies
  __amdgpu_buffer_rsrc_t wsrc[WI];
#pragma unroll
  for (int i = 0; i < WI; i++) {
    const int blk = min(bx * L::kBlocks + (wave * WI + i) / 4, a.total_blocks - 1);
    int b0;
    const int seg = block_seg(blk, b0);
    const void *w = seg == 0 ? w_0 : (seg == 1 ? w_1 : w_2);
    wsrc[i] = buffer_of((const char *)w + ((size_t)(blk - b0) * n_it_total + it_begin) * (size_t)kTileBytes + (wave * WI + i) % 4 * 1024);
  }
  // the X rows this wave copies: row segment rs = (t * 2 + g) * 32 + c holds the 64 bytes (32 k) of half g, its four 16-byte
  // pieces rotated by the row so that the fragment reads of eight consecutive rows touch all banks
  const int join = FOLD ? 0 : pinned(a.join);
  const uint32_t x_off0 = pinned(a.x_off[0]), x_off1 = pinned(a.x_off[1]);
  const __amdgpu_buffer_rsrc_t xsrc = buffer_of((const char *)(second ? x_1 : x_0) + (join ? 0 : (size_t)m0 * a.ldx * 2));
  uint32_t xoff[XI];
  int xk[XI];
#pragma unroll
  for (int i = 0; i < XI; i++) {
    const int rs = (wave * XI + i) * 16 + (lane >> 2);
    const int rc = rs & 31, rg = (rs >> 5) & 1, row = (rs >> 6) * 32 + rc;
    const int piece = (lane & 3) ^ ((rc >> 2) & 3);
    xk[i] = it_begin * 128 + rg * 64 + piece * 8;
    const int r = row < m_loc ? row : 0, r_all = m0 + r;
    xoff[i] = (uint32_t)(!join ? r : r_all < join ? r_all : r_all - join) * (uint32_t)a.ldx * 2u + (!join ? 0u : r_all < join ? x_off0 : x_off1);
  }
  auto load_w = [&](unsigned char *buf, int s, int i0, int i1) {
    s = min(s, n_stage - 1);                                  // past the end: the last stage again (never read)
#pragma unroll
    for (int i = i0; i < i1; i++) load_to_lds(wsrc[i], lane * 16, s * (kTileBytes / 2), buf + (wave * WI + i) * 1024);
  };
  auto load_x = [&](unsigned char *buf, int s) {
    s = min(s, n_stage - 1);
    const int ks = (s >> 1) * 128 + (s & 1) * 32;
#pragma unroll
    for (int i = 0; i < XI; i++) {
      const int k = xk[i] + ks;
      load_to_lds(xsrc, (int)(xoff[i] + (uint32_t)(k < a.in ? k : 0) * 2u), 0, buf + (wave * XI + i) * 1024);
    }
  };

  f32x16_t acc[WB][TB];
#pragma unroll
  for (int wb = 0; wb < WB; wb++)
#pragma unroll
    for (int t = 0; t < TB; t++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[wb][t][v] = 0.f;

  const int th = wave & (TW - 1), wq = wave / TW;
  const int xbase = th * TB * 4096 + (g * 32 + c) * 64, xsw = (c >> 2) & 3;
  const int wbase = wq * WB * 4096 + lane * 16;
  struct Frag { u32x4_t x[TB], w[WB]; };
  auto read = [&](Frag &f, const unsigned char *xb, const unsigned char *wb, int j) {
#pragma unroll
    for (int b = 0; b < WB; b++) f.w[b] = *(const u32x4_t *)(wb + wbase + b * 4096 + j * 1024);
#pragma unroll
    for (int t = 0; t < TB; t++) f.x[t] = *(const u32x4_t *)(xb + xbase + t * 4096 + ((j ^ xsw) * 16));
  };
  auto mul = [&](const Frag &f) {
#pragma unroll
    for (int wb = 0; wb < WB; wb++)
#pragma unroll
      for (int t = 0; t < TB; t++) mfma_step(acc[wb][t], f.x[t], f.w[wb], bf16_t{});
  };
  Frag f[2];
  // The order of a step: a fragment read of the next step behind each product, the copies behind the first ones.  In one bunch ahead
  // of the products they kept the LDS from both wavefronts of a SIMD at the same time (2048 x 28672 x 4096 467 -> 450 us, 1024 x 128256 x 4096
  // 951 -> 911).  The four products of the smallest tile's step are too few for that: its reads stay ahead (32 workgroups, K 2464 36 us against 39).
  constexpr bool kSpread = TB * WB > 4;
  auto ahead = [&]() __attribute__((always_inline)) { if constexpr (!kSpread) __builtin_amdgcn_sched_barrier(0); };
  auto spread = [&]() __attribute__((always_inline)) {
    if constexpr (kSpread) {
#pragma unroll
      for (int i = 0; i < TB * WB; i++) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);    // a matrix instruction
        if (i < TB + WB) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // an LDS read
        if (i >= 2) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);        // a copy
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto stage = [&](unsigned char *xc, unsigned char *wc, unsigned char *xn, unsigned char *wn, unsigned char *wp, int s) {
    // on entry f[0] = the fragments of step 0
#pragma unroll
    for (int j = 0; j < 3; j++) {
      read(f[(j + 1) & 1], xc, wc, j + 1);
      if (j == 0) load_w(wp, s + 2, 0, WI / 2);                // the copies spread over the steps
      if (j == 1) load_w(wp, s + 2, WI / 2, WI);
      ahead();
      mul(f[j & 1]);
      spread();
    }
    // every fragment of this stage is in registers, and this wave's share of the next one has arrived (only the W loads of the
    // stage after it may still be under way)
    __builtin_amdgcn_s_waitcnt(0x0070 | WI);                  // vmcnt(WI) lgkmcnt(0)
    wg_barrier();
    read(f[0], xn, wn, 0);
    load_x(xc, s + 2);
    ahead();
    mul(f[1]);
    spread();
  };

  f32x16_t sum[FOLD ? WB : 1][FOLD ? TB : 1];                 // FOLD: the finished ranges
  int range = 0, border = FOLD ? 2 * range_begin(1) : -1;     // stages before the next range begins
  auto fold = [&]() __attribute__((always_inline)) {
    if constexpr (FOLD) {
#pragma unroll
      for (int wb = 0; wb < WB; wb++)
#pragma unroll
        for (int t = 0; t < TB; t++)
#pragma unroll
          for (int v = 0; v < 16; v++) sum[wb][t][v] = range == 0 ? acc[wb][t][v] : sum[wb][t][v] + acc[wb][t][v];
    }
  };
  auto turn = [&](int done) __attribute__((always_inline)) {   // (a range is whole slabs, a multiple of four stages; the last one ends with the loop)
    if constexpr (FOLD) {
      if (done != border || done >= n_stage) return;
      fold();
#pragma unroll
      for (int wb = 0; wb < WB; wb++)
#pragma unroll
        for (int t = 0; t < TB; t++)
#pragma unroll
          for (int v = 0; v < 16; v++) acc[wb][t][v] = 0.f;
      range++;
      border = 2 * range_begin(range + 1);
    }
  };

  load_w(ws0, 0, 0, WI);
  load_x(xs0, 0);
  load_w(ws1, 1, 0, WI);
  load_x(xs1, 1);
  __builtin_amdgcn_s_waitcnt(0x0F70 | (WI + XI));             // stage 0 here
  wg_barrier();
  read(f[0], xs0, ws0, 0);
  int s = 0;
  for (; s + 6 <= n_stage; s += 6) {
    stage(xs0, ws0, xs1, ws1, ws2, s);
    stage(xs1, ws1, xs0, ws2, ws0, s + 1);
    turn(s + 2);
    stage(xs0, ws2, xs1, ws0, ws1, s + 2);
    stage(xs1, ws0, xs0, ws1, ws2, s + 3);
    turn(s + 4);
    stage(xs0, ws1, xs1, ws2, ws0, s + 4);
    stage(xs1, ws2, xs0, ws0, ws1, s + 5);
    turn(s + 6);
  }
  if (s < n_stage) {                                          // two or four stages are left: a K range is whole 128-k tiles
    stage(xs0, ws0, xs1, ws1, ws2, s);
    stage(xs1, ws1, xs0, ws2, ws0, s + 1);
    if (s + 2 < n_stage) {
      turn(s + 2);
      stage(xs0, ws2, xs1, ws0, ws1, s + 2);
      stage(xs1, ws0, xs0, ws1, ws2, s + 3);
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);                         // no copy into the LDS outlives the workgroup
  fold();

#pragma unroll
  for (int wb = 0; wb < WB; wb++) {
    const int blk = bx * L::kBlocks + wq * WB + wb;
    if (blk >= a.total_blocks) continue;
    if (swiglu) {
      const int f_ = rows_0, col = blk * 16 + (c & 15);
#pragma unroll
      for (int t = 0; t < TB; t++) {                          // one token block at a time: the exchange needs registers of its own
        const int i0 = (th * TB + t) * 32;
        const f32x16_t one[1] = {acc[wb][t]};
        swiglu_epilogue<1>(one, (bf16_t *)a.act + (size_t)(m0 + i0) * f_ + col, f_, col, col < f_, m_loc - i0, c, g);
        __builtin_amdgcn_sched_barrier(0);
      }
      continue;
    }
    int b0;
    const int seg = block_seg(blk, b0);
    const int rows = seg == 0 ? rows_0 : (seg == 1 ? rows_1 : rows_2);
    const int col0 = seg == 0 ? col_0 : (seg == 1 ? col_1 : col_2);
    const int row = (blk - b0) * 32 + c;
    if (row >= rows) continue;
    float *out = (second ? out_1 : out_0) + ((size_t)by * a.m_pad + m0 + th * TB * 32) * a.ldp;
    const uint32_t o0 = (uint32_t)(col0 + row);
#pragma unroll
    for (int t = 0; t < TB; t++)
#pragma unroll
      for (int v = 0; v < 16; v++) {
        const int i = t * 32 + 8 * (v >> 2) + 4 * g + (v & 3);
        if (th * TB * 32 + i < m_loc) out[o0 + (uint32_t)i * (uint32_t)a.ldp] = FOLD ? sum[FOLD ? wb : 0][FOLD ? t : 0][v] : acc[wb][t][v];
      }
  }
}

// Tiles of one shape.  Ids 8 apart run on one XCD: the token tiles of a weight tile follow each other there.
template <int TW, int TB, int WB, bool FOLD>
__global__ __launch_bounds__(kMmThreads, 2) void gemm_mm_kernel(GemmArgs a) {
  using L = MmTile<TW, TB, WB>;
  __shared__ __attribute__((aligned(1024))) unsigned char xs0[L::kX], xs1[L::kX], ws0[L::kW], ws1[L::kW], ws2[L::kW];
  const int per = 8 * a.m_tiles;
  const int q = ((int)blockIdx.x / per) * 8 + ((int)blockIdx.x % 8);
  const int mt = ((int)blockIdx.x % per) / 8;
  if (q >= a.grid_x * (FOLD ? 1 : a.n_split)) return;
  const int set_tiles = (a.m + L::kTok - 1) / L::kTok;        // tiles of the second set of rows follow the first set's
  const bool second = mt >= set_tiles;
  mm_tile_body<TW, TB, WB, FOLD>(a, q % a.grid_x, FOLD ? 0 : q / a.grid_x, second, (second ? mt - set_tiles : mt) * L::kTok, xs0, xs1, ws0, ws1, ws2);
}

// Measured against whole tiles only (us, launches of one shape): 2048 x 28672 x 4096 (3.5 rounds) 455 -> 432, 1024 x 57344 x 8192 841 -> 803, 1333 x
// 28672 x 4096 320 -> 300.  In a prompt of thousands of rows, where every launch runs into the power limit, less of it is left: whole requests 0.7 to 1 %.
// Tiles of 256 x 256 and, for what they would leave the chip half empty with, halves of 128 x 256: the tiles behind the last whole round
// of an XCD's 32 compute units, and a last token tile of up to 128 rows.  XCD x = id % 8 has the weight tiles (and K ranges) x, x + 8, ..; its
// list is every full token tile of each, in that order: n_big of them whole, the rest as pairs of halves, then the ragged ends.
__global__ __launch_bounds__(kMmThreads, 2) void gemm_mm_mixed_kernel(GemmArgs a) {
  using L = MmTile<2, 4, 2>;
  using H = MmTile<2, 2, 2>;
  static_assert(H::kW == L::kW && 2 * H::kTok == L::kTok, "a half is half the tokens of a tile");
  __shared__ __attribute__((aligned(1024))) unsigned char xs0[L::kX], xs1[L::kX], ws0[L::kW], ws1[L::kW], ws2[L::kW];
  const MmLists l = mm_lists(a.m, a.x2 ? 2 : 1, a.grid_x * a.n_split);
  const int x = (int)blockIdx.x % 8, j = (int)blockIdx.x / 8;
  const int n_q = (l.weight_tiles - x + 7) / 8, n_full = n_q * l.full;
  int ql, set, m0;
  const bool big = a.beside ? j % (l.full + l.ragged) < l.full : j < a.n_big;
  if (a.beside) {
    const int t = j % (l.full + l.ragged);
    ql = j / (l.full + l.ragged);
    if (ql >= n_q) return;
    set = big ? t / l.set_full : t - l.full;
    m0 = (big ? t % l.set_full : l.set_full) * L::kTok;
  } else if (big || j - a.n_big < 2 * (n_full - a.n_big)) {
    const int h = big ? 0 : j - a.n_big, t = big ? j : a.n_big + h / 2;
    if (t >= n_full) return;
    ql = t / l.full;
    const int tok = t % l.full;
    set = tok / l.set_full;
    m0 = (tok % l.set_full) * L::kTok + (h & 1) * H::kTok;
  } else {
    const int r = j - a.n_big - 2 * max(n_full - a.n_big, 0);
    if (r >= n_q * l.ragged) return;
    ql = r / l.ragged; set = r % l.ragged;
    m0 = l.set_full * L::kTok;
  }
  const int q = ql * 8 + x, bx = q % a.grid_x, by = q / a.grid_x;
  const bool second = __builtin_amdgcn_readfirstlane(set) != 0;
  if (big) mm_tile_body<2, 4, 2, false>(a, bx, by, second, m0, xs0, xs1, ws0, ws1, ws2);
  else mm_tile_body<2, 2, 2, false>(a, bx, by, second, m0, xs0, xs1, ws0, ws1, ws2);
}

// ---- fp32 storage ---------------------------------------------------------------------------------
// The fp32 configurations are small: a projection is a few hundred rows by a few hundred k, and a wavefront that walks all of
// K for a 32 x 32 tile (one v_mfma_f32_32x32x2 per two k, 64 cycles each) is what the launch waits for.  So the tile is
// 16 weight rows wide per MFMA (v_mfma_f32_16x16x4: no products for absent rows with up to 16 tokens), the four wavefronts of a
// workgroup split its K range by whole 64-k tiles (wavefront w takes tiles w, w + 4, ...), and their sums meet in the LDS once,
// in wavefront order.  Nothing is staged: a wavefront reads its own operands, the 16-byte pieces of a 16-token block and RB
// half weight blocks, one 64-k tile ahead.  The order of a row's sums depends on K and the split alone.
// Measured (MI355X), against 32 x 32 tiles with all of K in one wavefront: the projections of a 256-wide layer, up to 16 rows,
// 9.4 -> 3.4 us per launch.  Launches that fill the chip take gemm_f32_tiled_kernel below (same bits).
// Lane (r = lane % 16, kg = lane / 16) supplies row r and, in step jj of a tile, the four k of piece (g = kg % 2, j = 2 jj + kg / 2).
//
// KIND: the row kernel that makes x runs inside the launch (HeadKind).  At a 256-wide layer these kernels were a third of a forward's launches, 2 to 3 us each
// and as much again between them, for 16 KB of work.  Every workgroup makes the rows of its token block for itself, into the LDS (four wavefronts, four
// rows each; the weights of the first tile are requested before); the workgroups of the first weight block also store them and the residual rows.  The
// rotary table is filled by a workgroup per token block that has no weights.  Same operations in the same order as the row kernels: same bits.
// Request of the small fp32 model (66 launches a cycle -> 50) 4.54 -> 4.25 ms.
constexpr int kHeadCols = 512;                                // widest row
template <int RB, int KIND>
__global__ __launch_bounds__(kGemmThreads) void gemm_f32_kernel(GemmArgs a, HeadArg<KIND> head) {
  constexpr int E = RB * 4;                                   // sums per lane
  __shared__ float sums[kGemmWaves][E][kWave];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, kg = lane >> 4;
  const int tiles = (a.m + 15) / 16;                          // per set of rows
  const bool second = (int)blockIdx.z >= tiles;
  const int m0 = ((int)blockIdx.z - (second ? tiles : 0)) * 16, m_loc = min(a.m - m0, 16);
  if constexpr (KIND == kHeadEmbed || KIND == kHeadConcat) {
    if (blockIdx.x == gridDim.x - 1) {                        // the rotary table's workgroup
      if (blockIdx.y == 0)
        for (int n = tid; n < m_loc * head.rope.half; n += kGemmThreads) {
          const int i = m0 + n / head.rope.half, j = n % head.rope.half;
          head.rope.table[i * head.rope.half + j] = rope_entry(head.rope.pos[i], j, head.rope.half, head.rope.log2_theta);
        }
      return;
    }
  }
  const int by = blockIdx.y, blk = RB == 2 ? (int)blockIdx.x : (int)blockIdx.x >> 1, h0 = RB == 2 ? 0 : (int)blockIdx.x & 1;
  const int e0 = a.seg_blocks[0], e1 = e0 + (a.nseg > 1 ? a.seg_blocks[1] : 0);
  const int seg = blk < e0 ? 0 : (blk < e1 ? 1 : 2);
  const int b0 = seg == 0 ? 0 : (seg == 1 ? e0 : e1);
  const int seg_rows = seg == 0 ? a.seg_rows[0] : (seg == 1 ? a.seg_rows[1] : a.seg_rows[2]);
  const int seg_col0 = seg == 0 ? a.seg_col0[0] : (seg == 1 ? a.seg_col0[1] : a.seg_col0[2]);
  const void *seg_w = seg == 0 ? a.seg_w[0] : (seg == 1 ? a.seg_w[1] : a.seg_w[2]);
  constexpr int KI = 64;
  const int n_it_total = (a.in + KI - 1) / KI;
  const int it_begin = slab_begin(a, by) * kSlabIters;
  const int it_end = min(n_it_total, slab_begin(a, by + 1) * kSlabIters);

  const char *w0 = (const char *)seg_w + (size_t)(blk - b0) * n_it_total * kTileBytes + (((kg & 1) * 32 + r) * 16 + (kg >> 1) * 1024);
  const float *xbase = (const float *)(second ? a.x2 : a.x) + (size_t)m0 * a.ldx;
  const float *xrow = xbase + (size_t)(r < m_loc ? r : 0) * a.ldx, *erow = nullptr;
  if constexpr (KIND == kHeadConcat) {
    const int i = m0 + (r < m_loc ? r : 0);
    xrow = (const float *)head.feat + (size_t)(head.src_row ? head.src_row[i] : i) * head.d;
    erow = (const float *)head.embed + (size_t)head.token[i] * head.d - head.d;
  }
  constexpr bool kRows = KIND == kHeadSums || KIND == kHeadEmbed;
  constexpr int kXStride = kHeadCols + 4;                     // floats of a row in the LDS
  __shared__ __attribute__((aligned(16))) float xs[kRows ? 16 * kXStride : 4];
  f32x4_t acc[RB];
#pragma unroll
  for (int b = 0; b < RB; b++) acc[b] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  struct Tile { f32x4_t x[4], w[4][RB]; };
  const int n_tiles = max(0, (it_end - it_begin - wave + 3) / 4);   // of this wavefront
  auto load_w = [&](Tile &d, int s) {
    const char *wp = w0 + (size_t)(it_begin + wave + 4 * s) * kTileBytes;
#pragma unroll
    for (int jj = 0; jj < 4; jj++)
#pragma unroll
      for (int b = 0; b < RB; b++) d.w[jj][b] = *(const f32x4_t *)(wp + (h0 + b) * 256 + jj * 2048);
  };
  auto load_x = [&](Tile &d, int s) {
#pragma unroll
    for (int jj = 0; jj < 4; jj++) {
      int kk = (it_begin + wave + 4 * s) * KI + (kg & 1) * 32 + (2 * jj + (kg >> 1)) * 4;
      kk = kk < a.in ? kk : 0;                                // past K: meets a zero weight
      if constexpr (kRows) d.x[jj] = *(const f32x4_t *)(xs + (r < m_loc ? r : 0) * kXStride + kk);
      else if constexpr (KIND == kHeadConcat) d.x[jj] = *(const f32x4_t *)((kk < head.d ? xrow : erow) + kk);
      else d.x[jj] = *(const f32x4_t *)(xrow + kk);
    }
  };
  auto load = [&](Tile &d, int s) { load_w(d, s); load_x(d, s); };
  auto mul = [&](const Tile &d) {
#pragma unroll
    for (int jj = 0; jj < 4; jj++)
#pragma unroll
      for (int e = 0; e < 4; e++)
#pragma unroll
        for (int b = 0; b < RB; b++) acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(d.x[jj][e], d.w[jj][b][e], acc[b], 0, 0, 0);
  };
  Tile cur, nxt;
  if constexpr (kRows) {
    constexpr int NB = kHeadCols / 256;                       // a lane has columns 256 b + 4 lane .. + 3
    f32x4_t v[4][NB], nw[NB];
#pragma unroll
    for (int b = 0; b < NB; b++) {
      const int c = b * 256 + lane * 4, cc = c < head.d ? c : 0;
      if (b * 256 >= head.d) continue;
      nw[b] = head.norm_w != nullptr ? *(const f32x4_t *)((const float *)head.norm_w + cc) : f32x4_t{1.f, 1.f, 1.f, 1.f};
#pragma unroll
      for (int j = 0; j < 4; j++) {
        const int i = m0 + min(wave + 4 * j, m_loc - 1);
        if constexpr (KIND == kHeadEmbed) v[j][b] = *(const f32x4_t *)((const float *)head.embed + (size_t)head.token[i] * head.d + cc);
        else v[j][b] = *(const f32x4_t *)(head.part + (size_t)i * head.ldp + cc);
      }
    }
    if constexpr (KIND == kHeadSums) {
      f32x4_t res[4][NB];
#pragma unroll
      for (int b = 0; b < NB; b++) {
        const int c = b * 256 + lane * 4, cc = c < head.d ? c : 0;
        if (b * 256 >= head.d || !head.residual) continue;
#pragma unroll
        for (int j = 0; j < 4; j++) res[j][b] = *(const f32x4_t *)(head.h_in + (size_t)(m0 + min(wave + 4 * j, m_loc - 1)) * head.d + cc);
      }
      if (n_tiles > 0) load_w(cur, 0);
#pragma unroll
      for (int b = 0; b < NB; b++) {
        const int c = b * 256 + lane * 4, cc = c < head.d ? c : 0;
        if (b * 256 >= head.d) continue;
#pragma unroll
        for (int j = 0; j < 4; j++) {
          for (int sp = 1; sp < head.n_split; sp++)
            v[j][b] += *(const f32x4_t *)(head.part + ((size_t)sp * head.m_pad + m0 + min(wave + 4 * j, m_loc - 1)) * head.ldp + cc);
          if (head.residual) v[j][b] = res[j][b] + v[j][b];
        }
      }
    } else {
      if (n_tiles > 0) load_w(cur, 0);
    }
    const bool store = blockIdx.x == 0 && by == 0;
#pragma unroll
    for (int j = 0; j < 4; j++) {
      const int i = wave + 4 * j;
      if (i >= m_loc) continue;
      float scale = 1.f;
      if (head.norm_w != nullptr) {
        float t = 0.f;
#pragma unroll
        for (int b = 0; b < NB; b++)
          if (b * 256 < head.d) t += wave_sum(b * 256 + lane * 4 < head.d ? add_squares(0.f, v[j][b]) : 0.f);
        scale = norm_scale(t, head.d, head.eps);
      }
#pragma unroll
      for (int b = 0; b < NB; b++) {
        const int c = b * 256 + lane * 4;
        if (c >= head.d) continue;
        f32x4_t o = v[j][b];
        if (head.norm_w != nullptr) o = o * scale * nw[b];
        *(f32x4_t *)(xs + i * kXStride + c) = o;
        if (store) {
          *(f32x4_t *)(head.h_out + (size_t)(m0 + i) * head.d + c) = v[j][b];
          *(f32x4_t *)((float *)a.x + (size_t)(m0 + i) * a.ldx + c) = o;
        }
      }
    }
    __syncthreads();
    if (n_tiles > 0) load_x(cur, 0);
  } else {
    if (n_tiles > 0) load(cur, 0);
  }
  int s = 0;
  for (; s + 2 < n_tiles; s += 2) {
    load(nxt, s + 1);
    mul(cur);
    load(cur, s + 2);
    mul(nxt);
  }
  if (s + 1 < n_tiles) {
    load(nxt, s + 1);
    mul(cur);
    mul(nxt);
  } else if (s < n_tiles) {
    mul(cur);
  }

  // lane (r, kg) holds, for weight row r of half h0 + b, tokens 4 * kg + v
#pragma unroll
  for (int b = 0; b < RB; b++)
#pragma unroll
    for (int v = 0; v < 4; v++) sums[wave][b * 4 + v][lane] = acc[b][v];
  __syncthreads();
  auto total = [&](int e) { return ((sums[0][e][lane] + sums[1][e][lane]) + sums[2][e][lane]) + sums[3][e][lane]; };
  const int i = 4 * kg + wave;                                // wavefront w finishes v = w
  if (a.act != nullptr) {                                     // SwiGLU (RB == 2): half 0 = gate rows, half 1 = the up rows of the same columns
    if constexpr (RB == 2) {
      const int col = blk * 16 + r;
      const float g = total(wave), u = total(4 + wave);
      if (i < m_loc && col < seg_rows) ((float *)a.act)[(size_t)(m0 + i) * seg_rows + col] = silu_mul(g, u);
    }
    return;
  }
  float *out = (second ? a.part2 : a.part) + ((size_t)by * a.m_pad + m0) * a.ldp + seg_col0;
#pragma unroll
  for (int b = 0; b < RB; b++) {
    const int row = (blk - b0) * 32 + (h0 + b) * 16 + r;
    const float y = total(b * 4 + wave);
    if (i < m_loc && row < seg_rows) out[(size_t)i * a.ldp + row] = y;
  }
}

// ---- fp32 storage, launches that fill the chip ----------------------------------------------------------
// gemm_f32_kernel fetches (tokens + weight rows) * 4 bytes for 2 * tokens * weight rows operations, in half used lines: about ten operations per
// byte, and once the launch fills the chip the L2 limits it at about 60 TFLOP/s.  Here four wavefronts share a tile of 32 tokens x 64 weight
// rows (two by two, 16 x 32 each) whose operands are copied straight into the LDS, 32 k at a time into a ring of four, three ahead (in the LDS
// that two tiles of 64 k, one ahead, took: what a launch of few k tiles waited for); both keep the packed layout there, in which a fragment
// read touches every bank evenly.  Three workgroups fit a compute unit, so one's waits are covered by the others (tiles of 64 x 64, 64 x 128
// and 128 x 128 were slower: fewer wavefronts).  Bound: the fp32 matrix rate (150 TFLOP/s in a loop of nothing but these instructions).
// The bits are gemm_f32_kernel's: an fp32 MFMA is a chain of fused multiply-adds in the order of its k (both shapes, checked against
// fmaf), the 64-k tiles w, w + 4, ... of the K range have one accumulator, w = 0, 1, 2, 3 one after the other here, and the four sums are
// added up in that order.
// Measured (MI355X, us; gemm_f32_kernel before): 512 x 32000 x 4096 1966 -> 1097 (122 TFLOP/s), 1400 x 32000 x 1024 1083 -> 786, 512 x 12288 x
// 4096 588 -> 406, 300 x 5504 x 1024 53 -> 44.  The ring of halves against two whole tiles, then ragged tiles without padding: two sets of 129
// rows x 9000, K = 512 38.1 -> 36.0 -> 34.9, K = 2048 116.8 -> 112.4 -> 105.8; two of 512 x 9000 x 512 97.9 -> 92.6, of 256 x 4096 x 4096 160 -> 151.
constexpr int kF32Blocks = 2;                                 // 32-row weight blocks per workgroup
__global__ __launch_bounds__(kGemmThreads, 3) void gemm_f32_tiled_kernel(GemmArgs a) {
  constexpr int KI = 64, HB = kTileBytes / 2, WI = 2, LOADS = WI + 1;   // half a tile (32 k) of a block; 1 KB copies per wave and half: weights, all
  // (arrays of their own: see gemm_mm_kernel)
  __shared__ __attribute__((aligned(1024))) unsigned char b0[3 * HB], b1[3 * HB], b2[3 * HB], b3[3 * HB];   // the tokens' half tile, then the weight blocks'
  static_assert(kF32Blocks == 2 && HB == 4096, "eight weight pieces and four token pieces per half tile, for four wavefronts");
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, kg = lane >> 4, th = wave & 1, wh = wave >> 1;   // the wavefront's 16 tokens and its weight block
  // ids 8 apart run on one XCD: the token tiles of a weight tile follow each other there
  const int per = 8 * a.m_tiles;
  const int q = ((int)blockIdx.x / per) * 8 + ((int)blockIdx.x % 8);
  const int mt = ((int)blockIdx.x % per) / 8;
  if (q >= a.grid_x * a.n_split) return;
  const int bx = q % a.grid_x, by = q / a.grid_x;
  const int set_tiles = (a.m + 31) / 32;
  const bool second = mt >= set_tiles;
  const int m0 = (second ? mt - set_tiles : mt) * 32, m_loc = min(a.m - m0, 32);
  // up to 16 tokens: the wavefronts that would have the other 16 take the second half of the weight block instead of padding
  const bool narrow = m_loc <= 16 && a.act == nullptr;
  const int n_it_total = (a.in + KI - 1) / KI;
  const int it_begin = slab_begin(a, by) * kSlabIters;
  const int it_end = min(n_it_total, slab_begin(a, by + 1) * kSlabIters);

  const int e0 = a.seg_blocks[0], e1 = e0 + (a.nseg > 1 ? a.seg_blocks[1] : 0);
  auto seg_of = [&](int blk, int &b0) { const int s = blk < e0 ? 0 : (blk < e1 ? 1 : 2); b0 = s == 0 ? 0 : (s == 1 ? e0 : e1); return s; };
  // the 1 KB pieces this wave copies: of a weight tile as it is, of the X rows (piece j of row c, half g at j * 1024 + (g * 32 + c) * 16)
  __amdgpu_buffer_rsrc_t wsrc;
  {
    const int blk = min(bx * kF32Blocks + (wave >> 1), a.total_blocks - 1);
    int first;
    const int seg = seg_of(blk, first);
    const void *w = seg == 0 ? a.seg_w[0] : (seg == 1 ? a.seg_w[1] : a.seg_w[2]);
    wsrc = buffer_of((const char *)w + (size_t)(blk - first) * n_it_total * kTileBytes + (wave & 1) * 2048);
  }
  const __amdgpu_buffer_rsrc_t xsrc = buffer_of((const float *)(second ? a.x2 : a.x) + (size_t)m0 * a.ldx);
  const uint32_t xrow = (uint32_t)((lane & 31) < m_loc ? lane & 31 : 0) * (uint32_t)a.ldx * 4u;
  auto copy = [&](unsigned char *buf, int it, int half) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < WI; i++) load_to_lds(wsrc, lane * 16, it * kTileBytes + half * HB + i * 1024, buf + HB + (wave * WI + i) * 1024);
    const int k = it * KI + (lane >> 5) * 32 + (half * 4 + wave) * 4;   // past K: meets a zero weight
    load_to_lds(xsrc, (int)(xrow + (uint32_t)(k < a.in ? k : 0) * 4u), 0, buf + wave * 1024);
  };

  f32x4_t acc[2], sum[2];                                     // by half of the weight block
  acc[0] = acc[1] = sum[0] = sum[1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  struct Frag { f32x4_t x, w[2]; };                           // of step jj, as in gemm_f32_kernel
  const int xfrag = ((kg & 1) * 32 + (narrow ? 0 : th * 16) + r) * 16 + (kg >> 1) * 1024;
  const int wfrag = (1 + wh) * HB + ((kg & 1) * 32 + (narrow ? th * 16 : 0) + r) * 16 + (kg >> 1) * 1024, wfrag1 = narrow ? wfrag : wfrag + 256;
  auto read = [&](Frag &f, const unsigned char *buf, int jj) __attribute__((always_inline)) {
    f.w[0] = *(const f32x4_t *)(buf + wfrag + jj * 2048);
    f.w[1] = *(const f32x4_t *)(buf + wfrag1 + jj * 2048);
    f.x = *(const f32x4_t *)(buf + xfrag + jj * 2048);
  };
  auto mul = [&](const Frag &f) __attribute__((always_inline)) {
    if (narrow) {
#pragma unroll
      for (int e = 0; e < 4; e++) acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.x[e], f.w[0][e], acc[0], 0, 0, 0);
      return;
    }
#pragma unroll
    for (int e = 0; e < 4; e++)
#pragma unroll
      for (int b = 0; b < 2; b++) acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.x[e], f.w[b][e], acc[b], 0, 0, 0);
  };
  Frag f[2];
  // tile `it` of those of group w: it_begin + w, + 4, ...; the copies' tile is up to three halves ahead
  int w = 0, it = it_begin, left = 2 * (it_end - it_begin), cw = 0, cit = it_begin;
  auto copy_next = [&](unsigned char *buf, int half) __attribute__((always_inline)) {
    copy(buf, cit, half);
    if (half == 0) return;
    const bool turn = cit + 4 >= it_end;
    cw = turn ? cw + 1 : cw;
    cit = turn ? it_begin + cw : cit + 4;
  };
  // half `h` of a tile, in `cur`; the next half is in `next`, the third one from here goes to `free`.  FULL: there is one
  // (asked at run time in the loop, the compiler no longer knows how many copies are in flight and waits for too many)
  auto stage = [&](auto full, int h, unsigned char *cur, unsigned char *next, unsigned char *free) __attribute__((always_inline)) {
    // on entry f[0] = the fragments of step 0; nobody reads `free` any more
    constexpr bool FULL = decltype(full)::value;
    read(f[1], cur, 1);
    if (FULL || left > 3) copy_next(free, 1 - h);
    __builtin_amdgcn_sched_barrier(0);                        // the reads ahead of the products that hide them
    mul(f[0]);
    __builtin_amdgcn_sched_barrier(0);
    if (FULL || left > 1) {                                   // every fragment of this half is in registers, the next half has arrived
      if (FULL || left > 3) __builtin_amdgcn_s_waitcnt(0x0076);       // vmcnt(6) lgkmcnt(0)
      else if (left == 3) __builtin_amdgcn_s_waitcnt(0x0073);
      else __builtin_amdgcn_s_waitcnt(0x0070);
      wg_barrier();
      read(f[0], next, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    mul(f[1]);
    __builtin_amdgcn_sched_barrier(0);
    left--;
    if (h == 0) return;
    const bool turn = it + 4 >= it_end;                       // the group's last tile
    if (turn) {
#pragma unroll
      for (int b = 0; b < 2; b++) {
        // (a group without tiles adds its zero in gemm_f32_kernel)
#pragma unroll
        for (int v = 0; v < 4; v++) sum[b][v] = (w == 0 ? acc[b][v] : sum[b][v] + acc[b][v]) + (left ? -0.f : 0.f);
        acc[b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      }
    }
    w = turn ? w + 1 : w;
    it = turn ? it_begin + w : it + 4;
  };
  constexpr std::true_type full{};
  constexpr std::false_type rest{};
  static_assert(LOADS == 3, "the counts of the waits");
  copy_next(b0, 0);
  copy_next(b1, 1);
  if (left >= 8) {
    copy_next(b2, 0);
    __builtin_amdgcn_s_waitcnt(0x0F76);                       // vmcnt(6): all but the last two halves have arrived
    wg_barrier();
    read(f[0], b0, 0);
    do {
      stage(full, 0, b0, b1, b3);
      stage(full, 1, b1, b2, b0);
      stage(full, 0, b2, b3, b1);
      stage(full, 1, b3, b0, b2);
    } while (left >= 8);
  } else {
    if (left > 2) copy_next(b2, 0);
    __builtin_amdgcn_s_waitcnt(0x0F70);
    wg_barrier();
    read(f[0], b0, 0);
  }
  if (left) {
    stage(rest, 0, b0, b1, b3);
    stage(rest, 1, b1, b2, b0);
  }
  if (left) {
    stage(rest, 0, b2, b3, b1);
    stage(rest, 1, b3, b0, b2);
  }
  if (left) {
    stage(rest, 0, b0, b1, b3);
    stage(rest, 1, b1, b2, b0);
  }

  // lane (r, kg) holds, for weight row r of a half, tokens th * 16 + 4 * kg + v
  const int blk = bx * kF32Blocks + wh, i0 = (narrow ? 0 : th * 16) + 4 * kg;
  if (blk >= a.total_blocks) return;
  if (a.act != nullptr) {                                     // SwiGLU: half 0 = gate rows, half 1 = the up rows of the same columns
    const int f_ = a.seg_rows[0], col = blk * 16 + r;
#pragma unroll
    for (int v = 0; v < 4; v++)
      if (i0 + v < m_loc && col < f_) ((float *)a.act)[(size_t)(m0 + i0 + v) * f_ + col] = silu_mul(sum[0][v], sum[1][v]);
    return;
  }
  int first;
  const int seg = seg_of(blk, first);
  const int rows = seg == 0 ? a.seg_rows[0] : (seg == 1 ? a.seg_rows[1] : a.seg_rows[2]);
  const int col0 = seg == 0 ? a.seg_col0[0] : (seg == 1 ? a.seg_col0[1] : a.seg_col0[2]);
  float *out = (second ? a.part2 : a.part) + ((size_t)by * a.m_pad + m0) * a.ldp + col0;
#pragma unroll
  for (int b = 0; b < 2; b++) {
    if (narrow && b) break;
    const int row = (blk - first) * 32 + (narrow ? th : b) * 16 + r;
#pragma unroll
    for (int v = 0; v < 4; v++)
      if (i0 + v < m_loc && row < rows) out[(size_t)(i0 + v) * a.ldp + row] = sum[b][v];
  }
}

static hipError_t launch_f32_tiled(GemmArgs a, hipStream_t st) {
  a.m_tiles = (a.m + 31) / 32 * (a.x2 ? 2 : 1);
  a.grid_x = (a.total_blocks + kF32Blocks - 1) / kF32Blocks;
  const long long grid = ((long long)a.grid_x * a.n_split + 7) / 8 * 8 * a.m_tiles;
  if (grid > 0x7FFFFFFFll) return hipErrorInvalidValue;
  hipLaunchKernelGGL(gemm_f32_tiled_kernel, dim3((unsigned)grid), dim3(kGemmThreads), 0, st, a);
  return hipGetLastError();
}
// Which launches take it: more than 16 rows (up to 16 one pass over the weights does in gemm_f32_kernel) and 1024 workgroups of that kernel, four
// per compute unit.  us, gemm_f32_kernel / this one: 846 (48 rows, 512 x 9000) 12.5 / 12.9; 960 (80, 2048 x 6144) 30 / 39, (160, 1024 x 3072) 15.2 /
// 14.4; 1024 (17, 4096 x 4096, 4 splits) 20.7 / 18.3, (128, 2752 x 1024, 4 splits) 12.7 / 11.8; 1128 (64, 1024 x 9000) 25.3 / 22.5; 1204 (100, 1024 x 5504)
// 20.4 / 21.9; 1248 (200, 1024 x 3072) 18.2 / 21.9; 1344 (100, 2048 x 6144) 41.4 / 39.3; 1376 (128, 1024 x 5504) 23.7 / 22.2, (17, 4096 x 22016) 120 / 83;
// 2000 (17, 1024 x 32000) 39 / 24; beyond that up to 2.4 times as fast.  16 rows of 1024 x 32000 21.4 / 23.7.
// The copies into the LDS need 16-byte aligned sources, and the kernel's offsets inside a tile are 32-bit.
static bool f32_tiled_pays(const GemmArgs &a) {
  uintptr_t low = (uintptr_t)a.x | (uintptr_t)a.x2 | (uintptr_t)a.seg_w[0];
  if (a.nseg > 1) low |= (uintptr_t)a.seg_w[1];
  if (a.nseg > 2) low |= (uintptr_t)a.seg_w[2];
  if ((low & 15) || a.ldx % 4 || a.ldx < 0 || a.ldx >= (1 << 22) || a.in >= (1 << 22)) return false;
  const long long rows = (long long)a.m * (a.x2 ? 2 : 1);
  return rows > 16 && (long long)((a.m + 15) / 16) * (a.x2 ? 2 : 1) * a.total_blocks * a.n_split >= 1024;
}

// gemm_f32_kernel: half weight blocks while whole ones are few, or with up to 16 rows some more (then the weights' way counts and
// not the products).  us, whole / half: 96 workgroups (16 rows, 1024 x 3072) 5.6 / 4.6, 128 (16 rows, 2752 x 1024, 4 splits) 4.7 / 4.1, (32 rows, 1024 x
// 1024, 2 splits) 4.1 / 4.1; 192 (32 rows, 1024 x 3072) 5.7 / 6.8, 256 (32 rows, 2752 x 1024) 4.9 / 5.8; up to 16 rows 172 (one row, 1024 x 5504) 5.4 / 5.0, 282
// (one row, 1024 x 9000) 8.8 / 7.1, 384 (16 rows, 4096 x 12288) 34.3 / 35.3, 512 (16 rows, 4096 x 4096, 4 splits) 13.3 / 14.7.  More 16-token blocks per
// workgroup (2, 3, 4, 6) only lengthen it: 48 rows of 688 x 256 4.0 / 5.1 with two, 6.3 with three.
static bool f32_halves(const GemmArgs &a, int tiles) { return a.act == nullptr && (long long)a.total_blocks * a.n_split * tiles <= (a.m <= 16 ? 300 : 128); }
template <int KIND>
static hipError_t launch_f32_small(const GemmArgs &a, int tiles, const HeadArg<KIND> &head, hipStream_t st) {
  const int more = KIND == kHeadEmbed || KIND == kHeadConcat ? 1 : 0;   // the rotary table's workgroups
  if (f32_halves(a, tiles))
    hipLaunchKernelGGL((gemm_f32_kernel<1, KIND>), dim3(a.total_blocks * 2 + more, a.n_split, tiles), dim3(kGemmThreads), 0, st, a, head);
  else
    hipLaunchKernelGGL((gemm_f32_kernel<2, KIND>), dim3(a.total_blocks + more, a.n_split, tiles), dim3(kGemmThreads), 0, st, a, head);
  return hipGetLastError();
}
static hipError_t launch_f32(const GemmArgs &a, hipStream_t st, const GemmHead *head) {
  const int tiles = (a.m + 15) / 16 * (a.x2 ? 2 : 1);
  if (head != nullptr)
    return head->kind == kHeadSums ? launch_f32_small<kHeadSums>(a, tiles, *head, st)
           : head->kind == kHeadEmbed ? launch_f32_small<kHeadEmbed>(a, tiles, *head, st) : launch_f32_small<kHeadConcat>(a, tiles, *head, st);
  if (f32_tiled_pays(a)) return launch_f32_tiled(a, st);
  if (tiles > 65535) return hipErrorInvalidValue;
  return launch_f32_small<kHeadNone>(a, tiles, NoHead{}, st);
}
// One bf16 row: its K range in the LDS, sums of a row that eight wavefronts hold in registers, or an attention's parts (gemm_row_kernel's comment has both sides).
static bool row_takes_head(const GemmArgs &a, const GemmHead &h) {
  if (a.m != 1 || a.x2 != nullptr || a.fold || a.n_split < 1) return false;
  const int slabs = (a.in + gemm_k_per_slab(1) - 1) / gemm_k_per_slab(1);
  if (row_bytes(slabs / a.n_split, slabs % a.n_split) > kRowLds) return false;
  if (h.kind == kHeadParts) return a.in == h.merge.hq * h.merge.hd && h.merge.hd % 4 == 0 && ((uintptr_t)h.merge.part & 7) == 0;
  const uintptr_t low = (uintptr_t)a.x | (uintptr_t)h.part | (uintptr_t)h.h_in | (uintptr_t)h.h_out;
  return h.kind == kHeadSums && a.in == h.d && h.d % 4 == 0 && h.d <= kRowMaxCols && h.ldp % 4 == 0 && h.n_split >= 1 && (low & 15) == 0 &&
         ((uintptr_t)h.norm_w & 7) == 0;
}
// Whether a launch makes its own x: one bf16 row, and launches of gemm_f32_kernel over one set of up to 128 rows.  Rows of up to 256 columns always (us, two layers and their
// draft, 256 wide, launches of their own / this: draft of 4-row passes 157 / 139, of 10 367 / 342, of 16 507 / 480; verify and accept of 16 rows 97 / 91,
// 60 97 / 95, 128 107.5 / 105.5); of up to 512 with at most three rows a wavefront (512 wide: drafts of 4 rows 169.5 / 163, of 10 394 / 390, of 16 525 / 528; verify of one
// row 93.7 / 92, of 16 101.5 / 108, 60 109.5 / 115.5, 128 125.5 / 130).
bool gemm_takes_head(int dtype, const GemmArgs &a, const GemmHead &h) {
  if (dtype == 1) return row_takes_head(a, h);
  if (h.kind == kHeadParts) return false;
  if (dtype != 0 || h.kind == kHeadNone || a.m < 1 || a.m > kMaxNodes || a.x2 != nullptr || h.d % 4 || h.d > (a.m <= 12 ? kHeadCols : 256) || f32_tiled_pays(a))
    return false;
  if (h.kind != kHeadSums && (h.rope.table == nullptr || h.rope.half < 1)) return false;
  uintptr_t low = (uintptr_t)h.embed | (uintptr_t)h.feat | (uintptr_t)h.norm_w | (uintptr_t)h.part | (uintptr_t)h.h_in | (uintptr_t)h.h_out;
  if (h.kind == kHeadConcat) return (low & 15) == 0 && a.in == 2 * h.d;
  low |= (uintptr_t)a.x;
  return (low & 15) == 0 && a.in == h.d && a.ldx == h.d && (h.kind != kHeadSums || (h.ldp % 4 == 0 && h.n_split >= 1));
}

// ---- packing ---------------------------------------------------------------------------------
// One thread moves one 16-byte piece: dst piece index p = ((rb * n_it + it) * 8 + j) * 64 + lane.
template <typename T>
__global__ __launch_bounds__(256) void pack_weight_kernel(const T *src, int rows, int in, u32x4_t *dst, size_t n_pieces) {
  constexpr int EPL = GemmTraits<T>::kEpl;
  constexpr int KI = 2 * kLaneBytes / (int)sizeof(T);
  const int n_it = (in + KI - 1) / KI;
  for (size_t p = (size_t)blockIdx.x * 256 + threadIdx.x; p < n_pieces; p += (size_t)gridDim.x * 256) {
    const int lane = (int)(p & 63), j = (int)((p >> 6) & 7);
    const size_t tile = p >> 9;
    const int it = (int)(tile % n_it);
    const int rb = (int)(tile / n_it);
    const int row = rb * 32 + (lane & 31);
    const int k = it * KI + (lane >> 5) * (KI / 2) + j * EPL;
    u32x4_t v = {0u, 0u, 0u, 0u};
    if (row < rows && k < in) v = *(const u32x4_t *)(src + (size_t)row * in + k);     // in % EPL == 0: whole piece in range
    dst[p] = v;
  }
}

// The gate and up projections as ONE packed matrix: block b holds, in the row order of the layout above, the gate
// rows 16 b .. 16 b + 15 and then the up rows 16 b .. 16 b + 15 (zero rows past the last column), so that one wave
// owns both sums of a column and SwiGLU needs no second pass and no exchange between waves.
template <typename T>
__global__ __launch_bounds__(256) void pack_gate_up_kernel(const T *gate, const T *up, int rows, int in, u32x4_t *dst, size_t n_pieces) {
  constexpr int EPL = GemmTraits<T>::kEpl;
  constexpr int KI = 2 * kLaneBytes / (int)sizeof(T);
  const int n_it = (in + KI - 1) / KI;
  for (size_t p = (size_t)blockIdx.x * 256 + threadIdx.x; p < n_pieces; p += (size_t)gridDim.x * 256) {
    const int lane = (int)(p & 63), j = (int)((p >> 6) & 7);
    const size_t tile = p >> 9;
    const int it = (int)(tile % n_it);
    const int rb = (int)(tile / n_it);
    const int c = lane & 31;
    const int row = rb * 16 + (c & 15);
    const T *src = c < 16 ? gate : up;
    const int k = it * KI + (lane >> 5) * (KI / 2) + j * EPL;
    u32x4_t v = {0u, 0u, 0u, 0u};
    if (row < rows && k < in) v = *(const u32x4_t *)(src + (size_t)row * in + k);
    dst[p] = v;
  }
}

size_t packed_gate_up_bytes(int dtype, int rows, int in) {
  const int ki = gemm_k_per_iter(dtype);
  return (size_t)((rows + 15) / 16) * (size_t)((in + ki - 1) / ki) * kTileBytes;
}

hipError_t launch_pack_gate_up(int dtype, const void *gate, const void *up, int rows, int in, void *dst, hipStream_t st) {
  const int epl = dtype == 1 ? 8 : 4;
  if (rows < 1 || in < 1 || in % epl) return hipErrorInvalidValue;
  const size_t n_pieces = packed_gate_up_bytes(dtype, rows, in) / 16;
  const int blocks = (int)std::min<size_t>((n_pieces + 255) / 256, 65536);
  if (dtype == 1)
    hipLaunchKernelGGL(pack_gate_up_kernel<bf16_t>, dim3(blocks), dim3(256), 0, st, (const bf16_t *)gate, (const bf16_t *)up, rows, in,
                       (u32x4_t *)dst, n_pieces);
  else
    hipLaunchKernelGGL(pack_gate_up_kernel<float>, dim3(blocks), dim3(256), 0, st, (const float *)gate, (const float *)up, rows, in,
                       (u32x4_t *)dst, n_pieces);
  return hipGetLastError();
}

size_t packed_weight_bytes(int dtype, int rows, int in) {
  const int ki = gemm_k_per_iter(dtype);
  return (size_t)((rows + 31) / 32) * (size_t)((in + ki - 1) / ki) * kTileBytes;
}

hipError_t launch_pack_weight(int dtype, const void *src, int rows, int in, void *dst, hipStream_t st) {
  const int epl = dtype == 1 ? 8 : 4;
  if (rows < 1 || in < 1 || in % epl) return hipErrorInvalidValue;
  const size_t n_pieces = packed_weight_bytes(dtype, rows, in) / 16;
  const int blocks = (int)std::min<size_t>((n_pieces + 255) / 256, 65536);
  if (dtype == 1)
    hipLaunchKernelGGL(pack_weight_kernel<bf16_t>, dim3(blocks), dim3(256), 0, st, (const bf16_t *)src, rows, in, (u32x4_t *)dst, n_pieces);
  else
    hipLaunchKernelGGL(pack_weight_kernel<float>, dim3(blocks), dim3(256), 0, st, (const float *)src, rows, in, (u32x4_t *)dst, n_pieces);
  return hipGetLastError();
}

// The double-buffered slab exceeds the 64 KiB default for dynamic LDS from two token blocks on: raise the
// limit once per kernel, at context creation (never during a stream capture).
template <int TB>
static hipError_t init_tb() {
  const int lds = 2 * TB * 32 * kSlabStride;
  hipError_t e = hipSuccess;
  for (const void *f : {(const void *)gemm_stream_kernel<bf16_t, TB, false, kGemmWaves>, (const void *)gemm_stream_kernel<bf16_t, TB, true, kGemmWaves>,
                        (const void *)gemm_stream_kernel<bf16_t, TB, false, 8>, (const void *)gemm_stream_kernel<bf16_t, TB, true, 8>})
    if (e == hipSuccess) e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  return e;
}
hipError_t gemm_init() {
  // kernel attributes belong to the device's copy of the code: once per device, for the current device
  static bool done[64] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev >= 0 && dev < 64 && done[dev]) return hipSuccess;
  e = init_tb<1>();
  if (e == hipSuccess) e = init_tb<2>();
  if (e == hipSuccess) e = init_tb<3>();
  if (e == hipSuccess) e = init_tb<4>();
  if (dev >= 0 && dev < 64) done[dev] = e == hipSuccess;
  return e;
}

template <int TW, int TB, int WB, bool FOLD = false>
static hipError_t launch_mm_tile(GemmArgs a, hipStream_t st) {
  using L = MmTile<TW, TB, WB>;
  a.m_tiles = (a.m + L::kTok - 1) / L::kTok * (a.x2 ? 2 : 1);
  a.grid_x = (a.total_blocks + L::kBlocks - 1) / L::kBlocks;
  const dim3 grid((a.grid_x * (FOLD ? 1 : a.n_split) + 7) / 8 * 8 * a.m_tiles, 1);
  hipLaunchKernelGGL((gemm_mm_kernel<TW, TB, WB, FOLD>), grid, dim3(kMmThreads), 0, st, a);
  return hipGetLastError();
}
// A compute unit holds one workgroup, so a launch lasts as many rounds as its workgroups fill the 256 compute units.  A round
// of 256 x 256, 256 x 192 and 128 x 256 tiles (tokens x weight rows) takes 124, 90 and 62 us at K = 4096 and 37, 31 and 22 at 1024, of which about 6
// are filling and draining; the tile with the smallest product is taken, the larger one when they are close (it moves fewer bytes
// per product).  512 rows at the 7B shape: QKV (2 splits) 55 us with 256 x 192 against 58 and 74, gate/up 96 against 101 and 127,
// O (4 splits) 22 us with 128 x 256 against 23 and 26, LM head 124 us with 256 x 256 against 181 and 149.
// The 256 x 256 tile counts in whole rounds, though its last one may run in halves (mm_big_tiles).  Counted as it runs it would also be taken where it is
// slower than 128 x 256 (loss of 300 positions at vocabulary 32000 219 -> 226 us, of 257 226 -> 232, 300 rows of the 70B gate/up 364 -> 394) beside
// where it is faster (1333 rows of the 7B gate/up 249 -> 234, loss of 384 positions at vocabulary 128256 925 -> 900).
static float mm_us(int tile, int m, int sets, int blocks, int in, int n_split) {
  const int tok = tile == 2 ? 128 : 256, wb = tile == 1 ? 6 : 8;
  const float at4096 = tile == 0 ? 112.f : (tile == 1 ? 88.f : 64.f);
  const long long wgs = (long long)((m + tok - 1) / tok) * sets * ((blocks + wb - 1) / wb) * n_split;
  return (float)((wgs + 255) / 256) * (at4096 * (float)in / (4096.f * (float)n_split) + 6.f);
}
static int mm_tile(int m, int sets, int blocks, int in, int n_split) {
  int best = 0;
  float t = mm_us(0, m, sets, blocks, in, n_split);
  for (int tile = 1; tile < 3; tile++) {
    const float u = mm_us(tile, m, sets, blocks, in, n_split);
    if (u < 0.97f * t) { t = u; best = tile; }                // (launches of several rounds do not end exactly round by round)
  }
  return best;
}
void gemm_mm_tile(int m, int sets, int blocks, int in, int n_split, int *tokens, int *rows) {
  const int tile = mm_tile(m, sets, blocks, in, n_split);
  *tokens = tile == 2 ? 128 : 256; *rows = tile == 1 ? 192 : 256;
}
// The 256 x 256 tiles of an XCD that stay whole: all of them, or the whole rounds of its 32 compute units.  A whole tile takes tb, a half th
// (the times of mm_us); halves start wherever a compute unit is free.
static int mm_big_tiles(int m, int sets, int weight_tiles, int in, int n_split) {
  const MmLists l = mm_lists(m, sets, weight_tiles);
  const int n_q = (weight_tiles + 7) / 8, n_full = n_q * l.full, n_ragged = n_q * l.ragged;
  const float k = (float)in / (4096.f * (float)n_split), tb = 112.f * k + 6.f, th = 64.f * k + 6.f;
  auto us = [&](int big) {
    const int rounds = big / 32, rest = big % 32, free_cu = 32 - rest;
    int halves = n_ragged + 2 * (n_full - big);
    if (rest == 0) return rounds * tb + (float)((halves + 31) / 32) * th;
    halves -= free_cu;                                        // beside the last whole tiles
    return (rounds + 1) * tb + (float)(halves > 0 ? (halves + 31) / 32 : 0) * th;
  };
  const int whole = n_full / 32 * 32;
  return us(whole) < 0.97f * us(n_full) ? whole : n_full;
}
static hipError_t launch_mm_mixed(GemmArgs a, hipStream_t st) {
  const int sets = a.x2 ? 2 : 1;
  a.grid_x = (a.total_blocks + 7) / 8;
  const MmLists l = mm_lists(a.m, sets, a.grid_x * a.n_split);
  a.n_big = mm_big_tiles(a.m, sets, l.weight_tiles, a.in, a.n_split);
  const int n_q = (l.weight_tiles + 7) / 8;                   // (of XCD 0, the longest list)
  const int list = a.n_big + 2 * (n_q * l.full - a.n_big) + n_q * l.ragged;
  a.beside = a.join && l.ragged > 0 && l.full > 0 && a.n_big == n_q * l.full;
  hipLaunchKernelGGL(gemm_mm_mixed_kernel, dim3(8 * list), dim3(kMmThreads), 0, st, a);
  return hipGetLastError();
}
static float mm_xcd_us(int tile, int m, int blocks, int in, int ranges) {   // mm_us, with the rounds of the busiest XCD
  const int tok = tile == 2 ? 128 : 256, wb = tile == 1 ? 6 : 8;
  const float at4096 = tile == 0 ? 112.f : (tile == 1 ? 88.f : 64.f);
  const int per_xcd = ((blocks + wb - 1) / wb * ranges + 7) / 8 * ((m + tok - 1) / tok);
  return (float)((per_xcd + 31) / 32) * (at4096 * (float)in / (4096.f * (float)ranges) + 6.f);
}
// Tile of a folded launch: 256 x 192 or 128 x 256, whichever keeps the busiest XCD for less.  8B QKV of 2048 rows (6144 weight rows, K 4096): one
// round of 256 workgroups instead of one and a half of 384: 136 us a launch in a request -> 96 alone (107 as two sets of sums); 1333 rows 75 (81), 70B QKV of
// 1024 rows 170 (180).  A 4096-token prompt on 16 layers of the 8B widths 60.5 -> 59.6 ms a request, 1333 tokens on 8 layers 19.54 -> 19.30.
int gemm_fold_tile(int m, int blocks, int in) { return mm_xcd_us(1, m, blocks, in, 1) < 0.97f * mm_xcd_us(2, m, blocks, in, 1) ? 1 : 2; }
// Two sets of rows as one of twice the rows, its tiles running across the border: where that takes fewer tiles of 128 rows (a set's last, partly filled one
// is then the only one), the launch fills the chip all the same and the results of the second set follow those of the first.  A weight tile's ragged end
// then runs beside its whole tiles, so that the weights come from HBM once.  Row offsets are 32-bit.  Measured (us a loss, K = 4096 unless said, apart /
// joined): vocabulary 32000, 188 positions 145 / 134, 257 216 / 204, 300 223 / 210; 128256, 300, K = 2048 496 / 423, 700 (188 in the last chunk)
// 1666 / 1647; with the ragged ends behind all whole tiles 300 x 128256 took 470.  Vocabulary 1000, 188 positions, 12 tiles: 52.8 / 54.3, left apart,
// as are sets that would get a ragged end of a few rows where they have none (129 positions 137 / 137 to 150: its padding reads one row over and over).
static bool join_pays(int m, int blocks) {
  const long long tiles = (2ll * m + 127) / 128;
  if (m % 256 > 128 && m % 256 < 144) return false;
  return tiles < (m + 127) / 128 * 2ll && tiles * ((blocks + 7) / 8) >= 256;
}
static bool mm_joins(const GemmArgs &a) {
  if (a.x2 == nullptr || a.act != nullptr || a.n_split != 1 || !join_pays(a.m, a.total_blocks)) return false;
  if (a.part2 != a.part + (ptrdiff_t)a.m * a.ldp) return false;
  const uintptr_t x = (uintptr_t)a.x, x2 = (uintptr_t)a.x2, apart = x < x2 ? x2 - x : x - x2;
  return apart < (1u << 30) && 2ll * a.m * a.ldx + a.in < (1ll << 29);
}
static hipError_t launch_mm(const GemmArgs &args, hipStream_t st) {
  GemmArgs a = args;
  a.join = 0;
  if (mm_joins(a)) {
    const uintptr_t x = (uintptr_t)a.x, x2 = (uintptr_t)a.x2, base = std::min(x, x2);
    a.x_off[0] = (uint32_t)(x - base); a.x_off[1] = (uint32_t)(x2 - base);
    a.x = (const void *)base; a.x2 = nullptr; a.part2 = nullptr;
    a.join = a.m;
    a.m *= 2; a.m_pad = std::max(a.m_pad, a.m);
  }
  if (a.fold) return gemm_fold_tile(a.m, a.total_blocks, a.in) == 1 ? launch_mm_tile<4, 2, 3, true>(a, st) : launch_mm_tile<2, 2, 2, true>(a, st);
  switch (mm_tile(a.m, a.x2 ? 2 : 1, a.total_blocks, a.in, a.n_split)) {
    case 0: return launch_mm_mixed(a, st);
    case 1: return launch_mm_tile<4, 2, 3>(a, st);
    default: return launch_mm_tile<2, 2, 2>(a, st);
  }
}
// Whether m rows pay for folding the ranges instead of writing n_split sets of partial sums for `block` rows at a time.
// A set is written and read at about 8 TB/s (it stays in the memory-side cache).  us per layer of prefill, blocks -> fold: 7B shape, 1800 rows
// 1152 -> 1087, 4096 2594 -> 2493; 8B 2048 1290 -> 1213; 70B 1024 2072 -> 1997.  The 13B shape keeps the blocks: folded tiles of its 5120
// rows (20 per token tile) fall unevenly on the XCDs (1536 rows 1308 -> 1476 when folded), hence rounds by XCD.
bool gemm_fold_pays(int m, int rows, int in, int n_split, int block) {
  if (in >= (1 << 22) || rows >= (1 << 24)) return false;     // as mm_takes
  const int blocks = (rows + 31) / 32;
  const float set_us = (float)m * (float)rows * (8.f / 8e6f);
  float split_us = (float)n_split * set_us;
  for (int r0 = 0; r0 < m; r0 += block) {
    const int n = std::min(block, m - r0);
    split_us += mm_xcd_us(mm_tile(n, 1, blocks, in, n_split), n, blocks, in, n_split);
  }
  return mm_xcd_us(gemm_fold_tile(m, blocks, in), m, blocks, in, 1) + set_us < split_us;
}
// Copies into the LDS need 16-byte aligned sources, and the kernel's offsets inside a tile are 32-bit.
static bool mm_takes(const GemmArgs &a) {
  uintptr_t low = (uintptr_t)a.x | (uintptr_t)a.x2 | (uintptr_t)a.seg_w[0];
  if (a.nseg > 1) low |= (uintptr_t)a.seg_w[1];
  if (a.nseg > 2) low |= (uintptr_t)a.seg_w[2];
  return (low & 15) == 0 && a.ldx % 8 == 0 && a.ldx >= 0 && a.ldx < (1 << 22) && a.in < (1 << 22) && a.ldp < (1 << 24);
}

bool gemm_can_fold(const GemmArgs &a) { return a.act == nullptr && a.x2 == nullptr && mm_takes(a); }

template <int TB, bool PAIR>
static hipError_t launch_stream_tb(const GemmArgs &a, int waves, hipStream_t st) {
  constexpr size_t lds = (size_t)2 * TB * 32 * kSlabStride;
  static_assert(lds <= 160 * 1024, "the token blocks fit the LDS");
  const dim3 grid(a.grid_x, a.n_split), threads(waves * kWave);
  if (waves == 8) hipLaunchKernelGGL((gemm_stream_kernel<bf16_t, TB, PAIR, 8>), grid, threads, lds, st, a);
  else hipLaunchKernelGGL((gemm_stream_kernel<bf16_t, TB, PAIR, kGemmWaves>), grid, threads, lds, st, a);
  return hipGetLastError();
}
static int stream_blocks(int blocks, int n_split) {          // of the fullest workgroup when all compute units get one
  const int cap = std::max(1, 256 / n_split);
  return (blocks + cap - 1) / cap;
}
// Eight wavefronts share one X slab where that is worth it (the same sums in the same order):
//  * five to eight blocks per compute unit, any number of rows: one round of one workgroup each instead of a second, partly filled one of
//    workgroups of four.  Gate/up of 60 rows, K 4096, 1100 blocks 67.8 -> 50.2 us, 1500 73.8 -> 63.2, 2000 84.8 -> 82.3; K 8192, 1792 (70B) 152.7 -> 144.1,
//    ten rows 138.2 -> 136.5; 100 rows, 1500 blocks 96.7 -> 78.3;
//  * four on most compute units, up to 32 rows and K ranges up to 4096: four of the waves only stage, and the slab is there sooner.  1000 blocks,
//    K 4096, ten rows (7B LM head of the draft) 44.3 -> 41.7, 896 39.0 -> 37.5, 26 rows 40.0 -> 39.9; shorter ranges gain 6 to 9 %.  780 blocks 34.0 ->
//    35.7 (26 rows), K 5120 47.9 -> 49.3, 60 rows 41.3 -> 44.0;
//  * more than eight, more than 64 rows (a workgroup of four then has a compute unit to itself) and no more rounds x blocks: 100 rows, 4008 blocks 222 ->
//    193 (K 8192 434 -> 383; loss of 60 positions at that vocabulary 249 -> 219); 2300 144 -> 150, where two rounds of eight take the place of three of four.  Up to 64 rows two workgroups of four
//    share a compute unit: K 8192, 4008 blocks 335 -> 339 and 313 -> 324.
static int stream_waves(int tb, int blocks, int in, int n_split) {   // tb: 32-row token blocks
  const int units = blocks * n_split, per_wg = stream_blocks(blocks, n_split);
  const bool round8 = per_wg > kGemmWaves && per_wg <= 8;
  const bool stage8 = per_wg == kGemmWaves && tb == 1 && units >= 896 && (long long)in <= 4096ll * n_split;
  const bool slab8 = per_wg > 8 && tb >= 3 && 2 * ((per_wg + 7) / 8) <= (per_wg + 3) / 4;
  return round8 || stage8 || slab8 ? 8 : kGemmWaves;
}
void gemm_plan(int m, int sets, int blocks, int in, int n_split, int *waves, int *whole, int *tiles) {
  *waves = *whole = *tiles = 0;
  if ((long long)m * sets <= 128) { *waves = stream_waves((m * sets + 31) / 32, blocks, in, n_split); return; }
  if (sets == 2 && n_split == 1 && join_pays(m, blocks)) { m *= 2; sets = 1; }   // (where the sets' addresses allow it)
  if (mm_tile(m, sets, blocks, in, n_split) != 0) return;
  const int weight_tiles = (blocks + 7) / 8 * n_split;
  *tiles = (weight_tiles + 7) / 8 * mm_lists(m, sets, weight_tiles).full;
  *whole = mm_big_tiles(m, sets, weight_tiles, in, n_split);
}

template <int KIND, int WAVES>
static hipError_t launch_row(GemmArgs a, const GemmHead &head, hipStream_t st) {
  const int per_wg = std::min(WAVES, stream_blocks(a.total_blocks, a.n_split));   // blocks of a workgroup, on as many compute units as there are
  a.grid_x = (a.total_blocks + per_wg - 1) / per_wg;
  a.blk_per_wg = 1; a.blk_per_wave = a.grid_x;
  hipLaunchKernelGGL((gemm_row_kernel<KIND, WAVES>), dim3(a.grid_x, a.n_split), dim3(WAVES * kWave), row_bytes(a.slab_base, a.slab_rem), st, a, head);
  return hipGetLastError();
}

template <bool PAIR>
static hipError_t launch_stream(GemmArgs a, hipStream_t st) {
  const int tb = ((PAIR ? 2 * a.m : a.m) + 31) / 32;
  // Workgroups along the rows.  A compute unit sustains about 30 GB/s whatever the number of its waves, so what counts is
  // the largest number of blocks any workgroup streams.  With four blocks per workgroup the launch may leave compute
  // units idle (7B gate/up: 688 blocks = 172 workgroups); if the blocks fit in three, two or one per workgroup on at
  // most 256 workgroups (all splits together), the launch takes that form: wave w streams block x + w * grid_x and
  // the waves left without a block only help to stage the X slab (7B gate/up 36.1 -> 33.6 us, O 10.8 -> 10.0, down with
  // 4 splits 24.3 -> 20.3).  Otherwise four (or eight, stream_waves) adjacent blocks per workgroup: spreading without lowering the largest count
  // measured 1 - 4 % slower at the 13B shapes.
  const int per_wg = stream_blocks(a.total_blocks, a.n_split);
  const int waves = stream_waves(tb, a.total_blocks, a.in, a.n_split);
  if (per_wg < waves) {
    a.grid_x = (a.total_blocks + per_wg - 1) / per_wg;
    a.blk_per_wg = 1; a.blk_per_wave = a.grid_x;
  } else {
    a.grid_x = (a.total_blocks + waves - 1) / waves;
    a.blk_per_wg = waves; a.blk_per_wave = 1;
  }
  switch (tb) {
    case 1: return launch_stream_tb<1, PAIR>(a, waves, st);
    case 2: return launch_stream_tb<2, PAIR>(a, waves, st);
    case 3: return launch_stream_tb<3, PAIR>(a, waves, st);
    case 4: return launch_stream_tb<4, PAIR>(a, waves, st);
    default: return hipErrorInvalidValue;
  }
}

// Up to 128 rows in all the launch is bound by the weights, read once; a pair of row sets shares that one pass.
static hipError_t launch_bf16(const GemmArgs &a, hipStream_t st, const GemmHead *head) {
  const long long rows = (long long)a.m * (a.x2 ? 2 : 1);
  if (head != nullptr) return head->kind == kHeadSums ? launch_row<kHeadSums, 8>(a, *head, st) : launch_row<kHeadParts, kGemmWaves>(a, *head, st);
  if (a.fold && !gemm_can_fold(a)) return hipErrorInvalidValue;
  if (rows <= 128 && !a.fold) return a.x2 ? launch_stream<true>(a, st) : launch_stream<false>(a, st);
  if (mm_takes(a)) return launch_mm(a, st);
  for (int set = 0; set < (a.x2 ? 2 : 1); set++)               // any alignment: 128 rows at a time through the streaming kernel
    for (int m0 = 0; m0 < a.m; m0 += 128) {
      GemmArgs t = a;
      t.m = std::min(128, a.m - m0);
      t.x = (const char *)(set ? a.x2 : a.x) + (ptrdiff_t)m0 * a.ldx * (ptrdiff_t)sizeof(bf16_t);
      t.x2 = nullptr;
      if (a.act) t.act = (char *)a.act + (size_t)m0 * a.seg_rows[0] * sizeof(bf16_t);
      else t.part = (set ? a.part2 : a.part) + (size_t)m0 * a.ldp;
      const hipError_t e = launch_stream<false>(t, st);
      if (e != hipSuccess) return e;
    }
  return hipSuccess;
}

int gemm_k_per_iter(int dtype) { return dtype == 1 ? 128 : 64; }
int gemm_k_per_slab(int dtype) { return kSlabIters * gemm_k_per_iter(dtype); }

hipError_t launch_gemm(int dtype, const GemmArgs &args, hipStream_t st, const GemmHead *head) {
  GemmArgs a = args;
  if (head != nullptr && !gemm_takes_head(dtype, a, *head)) return hipErrorInvalidValue;
  { hipError_t e = gemm_init(); if (e != hipSuccess) return e; }
  if (a.m < 1 || a.m_pad < a.m || a.nseg < 1 || a.nseg > 3 || a.n_split < 1 || a.in < 1) return hipErrorInvalidValue;
  if (a.n_split > (a.in + gemm_k_per_slab(dtype) - 1) / gemm_k_per_slab(dtype)) return hipErrorInvalidValue;   // no empty split
  // SwiGLU mode: the one gate/up matrix, 16 columns per block, whole K (the activation is not linear)
  if (a.act != nullptr && (a.nseg != 1 || a.n_split != 1 || a.x2 != nullptr || a.seg_blocks[0] != (a.seg_rows[0] + 15) / 16))
    return hipErrorInvalidValue;
  const int slabs = (a.in + gemm_k_per_slab(dtype) - 1) / gemm_k_per_slab(dtype);
  const uint64_t inv = ~0ull / (uint64_t)a.n_split + 1;       // ceil(2^64 / n_split); 0 for n_split = 1
  a.slab_base = slabs / a.n_split; a.slab_rem = slabs % a.n_split;
  a.split_hi = (uint32_t)(inv >> 32); a.split_lo = (uint32_t)inv;
  return dtype == 1 ? launch_bf16(a, st, head) : launch_f32(a, st, head);
}

}  // namespace spec
