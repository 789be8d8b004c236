// Shared device helpers for the gfx950 kernels: storage types, conversions,
// wavefront (64-lane) reductions.  Nothing here is shared with the CPU oracle.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace spec {

constexpr int kWave = 64;

// bfloat16 kept as raw bits; arithmetic is always done in fp32.
struct bf16_t { uint16_t v; };

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t b) { return __uint_as_float(b << 16); }
__device__ __forceinline__ uint16_t f32_to_bf16_bits(float f) {   // round to nearest, ties to even (v_cvt_pk_bf16_f32)
  return __builtin_bit_cast(uint16_t, (__bf16)f);
}
// two floats -> two bf16 in one dword (lo in the low half), one hardware conversion
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  typedef __attribute__((ext_vector_type(2))) float f2_t;
  typedef __attribute__((ext_vector_type(2))) __bf16 b2_t;
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2_t{lo, hi}, b2_t));
}
__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(bf16_t x) { return bf16_bits_to_f32(x.v); }
template <typename T> __device__ __forceinline__ T from_f32(float x);
template <> __device__ __forceinline__ float from_f32<float>(float x) { return x; }
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float x) { bf16_t r; r.v = f32_to_bf16_bits(x); return r; }

// SwiGLU of one (gate, up) pair: silu(g) * u with silu(g) = g / (1 + e^-g), through the hardware's exp2 and reciprocal
// (about 1 ulp each; the result is rounded to the storage type afterwards).  Every kernel that forms the activation
// uses this one expression.
__device__ __forceinline__ float silu_mul(float g, float u) {
  const float e = __builtin_amdgcn_exp2f(g * -1.4426950408889634f);      // e^-g; large |g|: 0 or +inf, both give the right limit
  return g * __builtin_amdgcn_rcpf(1.0f + e) * u;
}

// Rotary embedding of the plane (a, b) = (dim j, dim j + hd/2) by (cos, sin).  Contraction into fused multiply-adds is
// switched off here: which product the compiler would fuse depends on the surrounding code, and every kernel that
// rotates the same inputs has to get the same bits.
__device__ __forceinline__ float rope_first(float a, float b, float2 cs) {
#pragma clang fp contract(off)
  const float x = a * cs.x, y = b * cs.y;
  return x - y;
}
__device__ __forceinline__ float rope_second(float a, float b, float2 cs) {
#pragma clang fp contract(off)
  const float x = b * cs.x, y = a * cs.y;
  return x + y;
}

// A store of a result that the NEXT kernel reads (on other XCDs), written through to device scope right away
// instead of staying dirty in this XCD's L2 until the end-of-kernel write-back.  Pays for the GEMM's partial sums
// (the reducing kernel that follows starts ~1 % of a cycle earlier, summed over a forward); the same for the row
// kernels changes nothing and for the attention partials, many small stores per lane, it costs 7 % of a verify.
__device__ __forceinline__ void store_through(float *p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void store_through(uint32_t *p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// What the lane `lane ^ O` holds, for a butterfly that goes through O = 32, 16, 8, 4, 2, 1 in this order, on the vector unit alone (a
// shuffle is a round trip through the LDS, about 100 cycles each: six of them were a third of a small row kernel's arithmetic).  O = 4 takes the
// lane 4 before in the row of 16, which after the steps before holds the same as lane ^ 4.  Needs all 64 lanes active.
template <int CTRL> __device__ __forceinline__ int dpp_i32(int x) { return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, true); }
template <int CTRL> __device__ __forceinline__ float dpp_f32(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true));
}
template <int O> __device__ __forceinline__ int butterfly(int x) {
  if constexpr (O >= 16) {                                    // the two halves (rows) swap: one result holds the lower one's, the other the upper one's
    const bool upper = (threadIdx.x & O) != 0;
    if constexpr (O == 32) { const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false); return upper ? r[0] : r[1]; }
    else { const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false); return upper ? r[0] : r[1]; }
  } else {
    return dpp_i32<(O == 8 ? 0x128 : O == 4 ? 0x124 : O == 2 ? 0x4E : 0xB1)>(x);   // row_ror 8, row_ror 4, quad_perm [2,3,0,1], [1,0,3,2]
  }
}
// Butterfly reductions over the 64 lanes of a wavefront; every lane gets the result.
// The exchange pattern is fixed, so the result does not depend on the data.  (f is commutative: of a swap's two results either order will do.)
template <typename F> __device__ __forceinline__ int wave_reduce(int x, F f) {
  { const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false); x = f(r[0], r[1]); }
  { const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false); x = f(r[0], r[1]); }
  x = f(x, butterfly<8>(x));
  x = f(x, butterfly<4>(x));
  x = f(x, butterfly<2>(x));
  return f(x, butterfly<1>(x));
}
__device__ __forceinline__ float wave_sum(float x) {
  return __int_as_float(wave_reduce(__float_as_int(x), [](int a, int b) { return __float_as_int(__int_as_float(a) + __int_as_float(b)); }));
}
__device__ __forceinline__ float wave_max(float x) {
  return __int_as_float(wave_reduce(__float_as_int(x), [](int a, int b) { return __float_as_int(fmaxf(__int_as_float(a), __int_as_float(b))); }));
}
__device__ __forceinline__ int wave_min_i(int x) { return wave_reduce(x, [](int a, int b) { return min(a, b); }); }
__device__ __forceinline__ int wave_sum_i(int x) { return wave_reduce(x, [](int a, int b) { return a + b; }); }

// Order-independent reductions (max, min) without LDS traffic: four DPP exchanges inside each row of 16
// lanes (xor 1, xor 2, mirror within 8, mirror within 16), then the four row results are read lane by lane.
// Needs all 64 lanes active.  Every lane gets the result.
__device__ __forceinline__ float wave_max_dpp(float x) {
  x = fmaxf(x, dpp_f32<0xB1>(x));     // quad_perm [1,0,3,2]
  x = fmaxf(x, dpp_f32<0x4E>(x));     // quad_perm [2,3,0,1]
  x = fmaxf(x, dpp_f32<0x141>(x));    // row_half_mirror
  x = fmaxf(x, dpp_f32<0x140>(x));    // row_mirror
  const int b = __float_as_int(x);
  return fmaxf(fmaxf(__int_as_float(__builtin_amdgcn_readlane(b, 0)), __int_as_float(__builtin_amdgcn_readlane(b, 16))),
               fmaxf(__int_as_float(__builtin_amdgcn_readlane(b, 32)), __int_as_float(__builtin_amdgcn_readlane(b, 48))));
}
__device__ __forceinline__ int wave_min_dpp(int x) {
  x = min(x, dpp_i32<0xB1>(x));
  x = min(x, dpp_i32<0x4E>(x));
  x = min(x, dpp_i32<0x141>(x));
  x = min(x, dpp_i32<0x140>(x));
  return min(min(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16)),
             min(__builtin_amdgcn_readlane(x, 32), __builtin_amdgcn_readlane(x, 48)));
}

// (value, index) pair ordered by larger value first, then lower index.
struct ValIdx { float v; int i; };
__device__ __forceinline__ bool better(float v, int i, float v2, int i2) { return v > v2 || (v == v2 && i < i2); }
template <int O> __device__ __forceinline__ void best_step(ValIdx &a) {
  const float ov = __int_as_float(butterfly<O>(__float_as_int(a.v)));
  const int oi = butterfly<O>(a.i);
  if (better(ov, oi, a.v, a.i)) { a.v = ov; a.i = oi; }
}
__device__ __forceinline__ ValIdx wave_best(ValIdx a) {
  best_step<32>(a); best_step<16>(a); best_step<8>(a); best_step<4>(a); best_step<2>(a); best_step<1>(a);
  return a;
}

// The same order as one unsigned 64-bit key (larger key = earlier): the value mapped monotonically to
// unsigned (-0 folded into +0), then the complemented index.  An empty entry (index INT_MAX) gets key 0,
// below every real entry.
__device__ __forceinline__ uint64_t order_key(float v, int i) {
  if (i == 0x7FFFFFFF) return 0ull;
  uint32_t u = __float_as_uint(v + 0.f);
  u ^= (u >> 31) ? 0xFFFFFFFFu : 0x80000000u;
  return ((uint64_t)u << 32) | (uint32_t)(0x7FFFFFFF - i);
}
// Number of keys ordered before key `k` held at list position `me`: larger keys, and equal keys (empty
// entries) at earlier positions.  `keys` is in LDS, 16-byte aligned, n2 (even) entries, zero-padded.
__device__ __forceinline__ int key_rank(const uint64_t *keys, int n2, uint64_t k, int me) {
  typedef __attribute__((ext_vector_type(2))) uint64_t u64x2_t;
  int rank = 0;
#pragma unroll 4
  for (int o = 0; o < n2; o += 2) {
    const u64x2_t kk = *(const u64x2_t *)(keys + o);
    rank += (kk.x > k || (kk.x == k && o < me)) ? 1 : 0;
    rank += (kk.y > k || (kk.y == k && o + 1 < me)) ? 1 : 0;
  }
  return rank;
}

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;

// Dynamic LDS beyond 64 KB, once per device: the attribute belongs to the device's copy of the code.
inline hipError_t allow_lds(const void *kernel, int bytes, bool (&done)[64]) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess || (dev >= 0 && dev < 64 && done[dev])) return e;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess && dev >= 0 && dev < 64) done[dev] = true;
  return e;
}

// ---- shared by the attention kernels ----
// Maximum over the lanes l and l ^ 32, in both, without the LDS round trip of a shuffle
__device__ __forceinline__ float max_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
// Value rows in the LDS: HD * 2 bytes a row, its 64-byte chunks permuted by the row so that the four rows a column read takes at a time
// lie in different banks.
template <int HD> __device__ __forceinline__ int value_chunk(int row, int chunk) { return chunk ^ (HD == 128 ? row & 3 : (row >> 1) & 1); }
template <int HD> __device__ __forceinline__ int value_piece(int row, int piece) { return row * HD * 2 + value_chunk<HD>(row, piece >> 2) * 64 + (piece & 3) * 16; }
// V^T fragments (A operand) out of them, by the LDS's transposing read (of the 4 x 16 matrix of 16-bit values whose row r the lanes 4 r .. 4 r + 3 of
// sixteen point at, lane i gets column i): lane (c, g) has dim db * 32 + c at keys first + 4 g + {0 .. 3, 8 .. 11}.
template <int HD> __device__ __forceinline__ int value_lane(int lane) {   // for db = 0, first = 0; db: ^ 64 db, first: a multiple of 16 rows further on
  const int row = 4 * (lane >> 5) + ((lane & 15) >> 2);
  return row * HD * 2 + value_chunk<HD>(row, 0) * 64 + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
}
typedef __attribute__((ext_vector_type(4))) short s16x4_t;
__device__ __forceinline__ u32x2_t read_columns(const unsigned char *p) {
  return __builtin_bit_cast(u32x2_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t *)p));
}
template <int HD> __device__ __forceinline__ u32x4_t value_fragment(const unsigned char *v_lds, int at, int db, int first) {
  const unsigned char *p = v_lds + (at ^ 64 * db) + first * HD * 2;
  const u32x2_t v0 = read_columns(p), v1 = read_columns(p + 8 * HD * 2);
  return u32x4_t{v0.x, v0.y, v1.x, v1.y};
}

// ---- merge of an attention's parts ----
// Scores are kept in units of log2: the launch's scale holds 1/sqrt(hd) * log2(e), and every weight is a power of two taken by the hardware.
__device__ __forceinline__ float exp2_(float x) { return __builtin_amdgcn_exp2f(x); }

// The merge of a row's parts, in ascending order and the tail last: (reference m, sum l, outputs o) of part after part go into the row's.  The row's
// reference moves only when a part's exceeds it by more than kRefSlack: until then weights are up to 2^kRefSlack, harmless in fp32, and the
// sums are left alone.  The final division cancels the choice.  step() returns what the row's sums are to be multiplied by before the part
// is added with weight w.
constexpr float kRefSlack = 8.f;
struct RowMerge {
  float m = -INFINITY, l = 0.f;
  __device__ __forceinline__ float step(float m_part, float l_part, float &w) {
    const bool move = m_part > m + kRefSlack;                  // also the first part
    const float m_new = move ? m_part : m;
    const float turn = move ? exp2_(m - m_new) : 1.f;
    m = m_new;
    w = exp2_(m_part - (m_new == -INFINITY ? 0.f : m_new));     // (a part whose scores are all -inf weighs nothing)
    l = fmaf(l_part, w, l * turn);
    return turn;
  }
};

// ---- RMSNorm rows and the rotary table: shared by every kernel that forms them (the same operations in the same order, so the bits do not depend on
// which does).  Virtual thread t of kNormThreads owns the 4-column groups t, t + kNormThreads, ..; its squares are added up in this order, then
// over the wavefronts of 64 virtual threads (wave_sum), then over these in ascending order.
constexpr int kNormThreads = 1024;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
__device__ __forceinline__ float add_squares(float ss, f32x4_t v) {
  float q = __builtin_fmaf(v.x, v.x, v.y * v.y);
  q = __builtin_fmaf(v.z, v.z, q);
  return ss + __builtin_fmaf(v.w, v.w, q);
}
__device__ __forceinline__ float norm_scale(float sum, int d, float eps) { return 1.0f / sqrtf(sum / (float)d + eps); }
template <typename T> __device__ __forceinline__ f32x4_t load4(const T *p);
template <> __device__ __forceinline__ f32x4_t load4<float>(const float *p) { return *(const f32x4_t *)p; }
template <> __device__ __forceinline__ f32x4_t load4<bf16_t>(const bf16_t *p) {
  const uint2 u = *(const uint2 *)p;
  return f32x4_t{__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xFFFF0000u), __uint_as_float(u.y << 16),
                 __uint_as_float(u.y & 0xFFFF0000u)};
}
// (cos, sin) of pos * theta^(-j/half), the angle formed in double so that large positions keep their phase
__device__ __forceinline__ float2 rope_entry(int pos, int j, int half, double log2_theta) {
  const double inv = exp2(-(double)j / (double)half * log2_theta);
  const double ang = (double)pos * inv;
  double s, c;
  sincos(ang, &s, &c);
  return make_float2((float)c, (float)s);
}

// Four rotary planes (a: their first dims, b: their partners `half` further on) of a row from the projection's partial sums p; rope: the planes' (cos, sin).  Not
// turned: the sums alone.  All loads first, up to NS splits (absent ones read split 0 again and are left out).
struct RotaryPlanes { f32x4_t a, b; };
template <int NS>
__device__ __forceinline__ RotaryPlanes rotary_planes(const float *p, int n_split, size_t split_stride, const float2 *rope, int half, bool turned) {
  const f32x4_t *cs = (const f32x4_t *)rope;
  const f32x4_t cs0 = cs[0], cs1 = cs[1];                     // of planes j, j + 1 and j + 2, j + 3
  f32x4_t pa[NS], pb[NS];
#pragma unroll
  for (int s = 0; s < NS; s++) {
    const float *q = p + (size_t)(s < n_split ? s : 0) * split_stride;
    pa[s] = *(const f32x4_t *)q; pb[s] = *(const f32x4_t *)(q + half);
  }
  RotaryPlanes x{pa[0], pb[0]};
#pragma unroll
  for (int s = 1; s < NS; s++)
    if (s < n_split) { x.a += pa[s]; x.b += pb[s]; }
  for (int s = NS; s < n_split; s++) { x.a += *(const f32x4_t *)(p + (size_t)s * split_stride); x.b += *(const f32x4_t *)(p + (size_t)s * split_stride + half); }
  if (turned) {
    const float2 c[4] = {{cs0.x, cs0.y}, {cs0.z, cs0.w}, {cs1.x, cs1.y}, {cs1.z, cs1.w}};
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const float u = rope_first(x.a[e], x.b[e], c[e]), v = rope_second(x.a[e], x.b[e], c[e]);
      x.a[e] = u; x.b[e] = v;
    }
  }
  return x;
}

// Block-wide sum for blocks of up to 16 waves; `sh` needs 16 floats.  Fixed order.
__device__ __forceinline__ float block_sum(float x, float *sh) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  x = wave_sum(x);
  __syncthreads();
  if (lane == 0) sh[w] = x;
  __syncthreads();
  float t = 0.f;
  for (int i = 0; i < nw; i++) t += sh[i];
  return t;
}
__device__ __forceinline__ float block_max(float x, float *sh) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  x = wave_max(x);
  __syncthreads();
  if (lane == 0) sh[w] = x;
  __syncthreads();
  float t = sh[0];
  for (int i = 1; i < nw; i++) t = fmaxf(t, sh[i]);
  return t;
}
__device__ __forceinline__ ValIdx block_best(ValIdx a, float *shv, int *shi) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  a = wave_best(a);
  __syncthreads();
  if (lane == 0) { shv[w] = a.v; shi[w] = a.i; }
  __syncthreads();
  ValIdx t{shv[0], shi[0]};
  for (int i = 1; i < nw; i++) if (better(shv[i], shi[i], t.v, t.i)) { t.v = shv[i]; t.i = shi[i]; }
  return t;
}

}  // namespace spec
