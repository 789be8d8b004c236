// Tree attention for the decode path: each query row attends to the committed KV cache and
// to the nodes on its own root-to-node path.
//
// Row i sits at key position p = base + depth[i].  Key position q < base lives in cache
// slot q; position q >= base lives in slot base + anc[i][q - base], i.e. the row's own
// ancestors (anc == nullptr: a causal chain, slot q).  The keys of a row are therefore
// visited in POSITION order, which is exactly the order plain decoding visits them after
// the accepted nodes have been compacted to consecutive slots: the arithmetic of a row is
// a function of (its query, the key/value rows by position) only, so speculative and
// plain decoding agree bit for bit.
//
// Two code paths share one definition of the key order:
//
//  * vector path (attn_part_kernel): one wavefront handles (row, kv head, part of the key positions:
//    kAttnPart = 128 of them below position kAttnNear, kAttnFarPart beyond) and all G query heads that share the kv head; keys are taken 64 at a time,
//    lane = position offset for the scores (wave shuffles give the running max and sum of the
//    online softmax), then lane = output dim for P*V, which runs over the value rows staged in
//    LDS key by key in position order.  Used for fp32 storage, and for the TAIL
//    of every row in bf16 storage.
//
//  * matrix-core path (bulk workgroups of attn_hybrid_kernel, bf16 storage): the BULK of a row's keys, positions
//    [0, A(p)) with A(p) = 32 * floor(max(p - kMaxDepth, 0) / 32), lies in the committed cache
//    for every row of a tree (depth <= kMaxDepth), is the same key set for spec and plain decoding,
//    and is shared by all rows, so it runs as dense 32-key blocks on the MFMA units: S^T = K Q^T
//    and O^T = V^T P^T with v_mfma_f32_32x32x16_bf16, K/V blocks staged once in LDS for all rows
//    (V transposed on the way out), queries and probabilities split into bf16 hi + lo parts so
//    that they keep fp32-class accuracy.  The remaining positions [A(p), p] (16..47 keys: the end
//    of the cache plus the row's own path) take the vector path.  A(p) depends on the position
//    only, so a row is computed by the same instructions over the same key groups whether it is
//    alone or part of a tree.  A prompt of hundreds of rows takes a kernel of its own (attn_chain_kernel) that repeats
//    this arithmetic step by step, merge included: its rows have the bits they would have alone.
//
// Parts (fixed absolute boundaries: attn_part_begin; larger parts for far keys, where a long context would otherwise
// mean many partials to merge and many short workgroups) are merged per row in ascending order, the tail
// last, by attn_combine_kernel (RowMerge).  In the hybrid path the bulk and the tail are independent and run in ONE
// launch (different workgroups), so the chain per layer is two dependent kernels.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace spec {


template <int N, int I = 0, typename F>
__device__ __forceinline__ void unrolled(F &&f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    unrolled<N, I + 1>(f);
  }
}

template <typename T> struct Chunk;   // 16-byte chunk -> floats
template <> struct Chunk<float> {
  static constexpr int kEpl = 4;
  static __device__ __forceinline__ void unpack(const u32x4_t &c, float *f) {
    f[0] = __uint_as_float(c.x); f[1] = __uint_as_float(c.y); f[2] = __uint_as_float(c.z); f[3] = __uint_as_float(c.w);
  }
};
template <> struct Chunk<bf16_t> {
  static constexpr int kEpl = 8;
  static __device__ __forceinline__ void unpack(const u32x4_t &c, float *f) {
    f[0] = __uint_as_float(c.x << 16); f[1] = __uint_as_float(c.x & 0xFFFF0000u);
    f[2] = __uint_as_float(c.y << 16); f[3] = __uint_as_float(c.y & 0xFFFF0000u);
    f[4] = __uint_as_float(c.z << 16); f[5] = __uint_as_float(c.z & 0xFFFF0000u);
    f[6] = __uint_as_float(c.w << 16); f[7] = __uint_as_float(c.w & 0xFFFF0000u);
  }
};

// Orders this wavefront's LDS writes before its later LDS reads of other lanes' data.  The LDS executes
// one wavefront's operations in issue order, so only the compiler has to be kept from reordering them.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One wavefront: row i, kv head hk, part `part`.  `qs` and `vs` are this wavefront's own LDS areas ([G][HD]
// floats and 64 staged value rows); no workgroup barrier is used, so wavefronts of one workgroup may work on
// different items.
template <typename T> struct PartLds {
  static constexpr int vrow(int hd) { return hd * (int)sizeof(T) + 16; }   // +16: conflict-free row writes
};
// AHEAD: the next 64 keys' rows are requested before this 64's are used (a second set of registers: where few wavefronts run).
// emit(head of the group, reference, sum, outputs) takes the result.
template <typename T, int HD, int G, bool AHEAD, typename Emit>
__device__ __forceinline__ void attn_part_body(const AttnArgs &a, int i, int hk, int part, int lane, float (*qs)[HD],
                                               unsigned char *vs, Emit emit) {
  constexpr int EPL = Chunk<T>::kEpl;
  constexpr int DPL = HD / 64;                       // output dims per lane (contiguous)
  constexpr int VROW = PartLds<T>::vrow(HD);         // LDS bytes per staged value row
  const int base = a.base_ptr ? *a.base_ptr : a.base;  // device-resident when the launch is replayed from a graph
  const int p = base + a.depth[i];
  const int k_lo = attn_part_begin(part);
  const int k_hi = min(p + 1, attn_part_begin(part + 1));
  if (k_lo >= k_hi) return;

  const float *qrow = (const float *)a.q + ((size_t)i * a.hq + (size_t)hk * G) * HD;   // queries are fp32
  for (int e = lane; e < G * HD; e += 64) qs[e / HD][e % HD] = qrow[e];

  float m_run[G], l_run[G], o[G][DPL];
#pragma unroll
  for (int gh = 0; gh < G; gh++) {
    m_run[gh] = -INFINITY; l_run[gh] = 0.f;
#pragma unroll
    for (int dd = 0; dd < DPL; dd++) o[gh][dd] = 0.f;
  }
  const int *anc = a.anc ? a.anc + (size_t)i * kAncStride : nullptr;
  const size_t row_stride = (size_t)a.hkv * HD;
  const T *kbase = (const T *)a.kcache + (size_t)hk * HD;
  const T *vbase = (const T *)a.vcache + (size_t)hk * HD;

  struct Rows { u32x4_t k[HD / EPL], v[HD / EPL]; };
  auto load = [&](Rows &r, int kb) __attribute__((always_inline)) {
    // lane = key: this lane's key row and value row (all loads issued before anything is used);
    // lanes past the range re-read the last key of the range (initialised data; their weight is 0)
    const int kr = min(kb + lane, k_hi - 1);
    const int slot = kr < base ? kr : base + (anc ? anc[kr - base] : kr - base);
    const T *kptr = kbase + (size_t)slot * row_stride;
    const T *vptr = vbase + (size_t)slot * row_stride;
#pragma unroll
    for (int dc = 0; dc < HD / EPL; dc++) r.k[dc] = *(const u32x4_t *)(kptr + dc * EPL);
#pragma unroll
    for (int dc = 0; dc < HD / EPL; dc++) r.v[dc] = *(const u32x4_t *)(vptr + dc * EPL);
  };
  Rows now, next;
  load(now, k_lo);
  for (int kb = k_lo; kb < k_hi; kb += 64) {
    const bool valid = kb + lane < k_hi;
    if (AHEAD && kb + 64 < k_hi) load(next, kb + 64);
    const u32x4_t (&kc)[HD / EPL] = now.k, (&vc)[HD / EPL] = now.v;
    wave_lds_sync();                                   // qs written (first pass) / previous block's vs reads done
    float s[G];
#pragma unroll
    for (int gh = 0; gh < G; gh++) s[gh] = 0.f;
#pragma unroll
    for (int dc = 0; dc < HD / EPL; dc++) {
      float kf[EPL];
      Chunk<T>::unpack(kc[dc], kf);
#pragma unroll
      for (int gh = 0; gh < G; gh++)
#pragma unroll
        for (int e = 0; e < EPL; e++) s[gh] = fmaf(qs[gh][dc * EPL + e], kf[e], s[gh]);
    }
    // stage the value rows: row `lane` of vs
#pragma unroll
    for (int dc = 0; dc < HD / EPL; dc++) *(u32x4_t *)(vs + lane * VROW + dc * 16) = vc[dc];
    float pk[G];
#pragma unroll
    for (int gh = 0; gh < G; gh++) {
      const float sc = valid ? s[gh] * a.scale : -INFINITY;
      const float m_new = fmaxf(m_run[gh], wave_max(sc));
      const float corr = exp2_(m_run[gh] - m_new);       // first block: 2^-inf = 0
      pk[gh] = valid ? exp2_(sc - m_new) : 0.f;
      l_run[gh] = l_run[gh] * corr + wave_sum(pk[gh]);
#pragma unroll
      for (int dd = 0; dd < DPL; dd++) o[gh][dd] *= corr;
      m_run[gh] = m_new;
    }
    wave_lds_sync();                                   // value rows staged
    // lane = output dims lane*DPL ..: accumulate key by key in position order
    // Eight keys per step so that the LDS reads of a step are in flight together.  Lanes past the last
    // key hold weight 0 and a finite value row (a copy of the last key's), so rounding a step up to eight adds zeros.
    const int nk = min(64, k_hi - kb);
    const unsigned char *vcol = vs + lane * DPL * (int)sizeof(T);
    for (int k0 = 0; k0 < nk; k0 += 8) {
      float vv[8][DPL];
#pragma unroll
      for (int kk = 0; kk < 8; kk++)
#pragma unroll
        for (int dd = 0; dd < DPL; dd++) vv[kk][dd] = to_f32(*(const T *)(vcol + (k0 + kk) * VROW + dd * (int)sizeof(T)));
#pragma unroll
      for (int kk = 0; kk < 8; kk++)
#pragma unroll
        for (int gh = 0; gh < G; gh++) {
          const float w = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(pk[gh]), k0 + kk));
#pragma unroll
          for (int dd = 0; dd < DPL; dd++) o[gh][dd] = fmaf(w, vv[kk][dd], o[gh][dd]);
        }
    }
    if (kb + 64 < k_hi) {
      if constexpr (AHEAD) now = next;
      else load(now, kb + 64);
    }
  }
#pragma unroll
  for (int gh = 0; gh < G; gh++) emit(gh, m_run[gh], l_run[gh], o[gh]);
}

// The tail of a row in the hybrid path: positions [max(p - kMaxDepth, 0), p], at most kTailKeys = 16 keys,
// the end of the committed cache followed by the row's own path.  One wavefront per (row, kv head): four
// lanes share a key (each takes a quarter of the head dim for the score, summed over the quad in a fixed
// order), then lane = output dim for P*V over the value rows staged in LDS, key by key in position order.
// The result goes to the last part slot.
constexpr int kTailKeys = kMaxDepth + 1;
static_assert(kTailKeys * 4 == 64, "one wavefront = 16 keys x 4 lanes");
// The rotary planes j .. j + 3 of a head (columns col .. of the partial sums, the planes' partners HD / 2 further on) of row i from the QKV projection's partial sums
__device__ __forceinline__ RotaryPlanes raw_planes(const AttnRaw &r, int i, int col, int half, int j, bool turned) {
  return rotary_planes<4>(r.qkv + (size_t)i * r.ldp + col, r.n_split, r.split_stride, r.rope + (size_t)i * half + j, half, turned);
}
__device__ __forceinline__ uint2 pack4(f32x4_t v) { return uint2{pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w)}; }
// RAW: queries, key and value of the row come from the partial sums.  The row's own key and value go to own (LDS, the stored type, key first) and to the caches;
// all other keys are in the caches.  `store` = false discards the result.
template <typename T, int HD, int G, bool RAW = false>
__device__ __forceinline__ void attn_tail_body(const AttnArgs &a, int i, int hk, int lane, float (*qs)[HD],
                                               unsigned char *vs, bool store, T *own = nullptr) {
  constexpr int EPL = Chunk<T>::kEpl;
  constexpr int DPL = HD / 64;                       // output dims per lane (contiguous)
  constexpr int VROW = PartLds<T>::vrow(HD);
  constexpr int QD = HD / 4;                         // dims per lane of a key quad
  constexpr int QC = QD / EPL;                       // 16-byte chunks per lane
  const int base = a.base_ptr ? *a.base_ptr : a.base;
  const int p = base + a.depth[i];
  const int k_lo = bulk_end(p);
  const int kk = lane >> 2, qt = lane & 3;
  const int kq = k_lo + kk;
  const bool valid = kq <= p;
  const int *anc = a.anc ? a.anc + (size_t)i * kAncStride : nullptr;
  // lanes past position p re-read the row's own key (initialised data; their weight is 0)
  const bool mine = RAW && kq >= p;                  // the row's own key, out of the LDS (the address below is then only a valid one)
  const int kr = mine ? max(p - 1, 0) : valid ? kq : p;
  const int slot = kr < base ? kr : base + (anc ? anc[kr - base] : kr - base);
  const size_t row_stride = (size_t)a.hkv * HD;
  const T *kptr = (const T *)a.kcache + (size_t)slot * row_stride + (size_t)hk * HD + qt * QD;
  const T *vptr = (const T *)a.vcache + (size_t)slot * row_stride + (size_t)hk * HD + qt * QD;
  u32x4_t kc[QC], vc[QC];
#pragma unroll
  for (int dc = 0; dc < QC; dc++) kc[dc] = *(const u32x4_t *)(kptr + dc * EPL);
#pragma unroll
  for (int dc = 0; dc < QC; dc++) vc[dc] = *(const u32x4_t *)(vptr + dc * EPL);
  if constexpr (RAW) {
    static_assert(sizeof(T) == 2, "bf16 rows");
    constexpr int half = HD / 2, per_head = half / 4;
    T *const cache[2] = {(T *)a.kcache, (T *)a.vcache};
    const size_t at = ((size_t)a.raw.slot[i] * a.hkv + hk) * HD;
#pragma unroll
    for (int e0 = 0; e0 < (G + 2) * per_head; e0 += 64) {     // heads of the group, then the key, then the value
      const int e = e0 + lane, head = e / per_head, j = e % per_head * 4;
      if (e >= (G + 2) * per_head) continue;
      const int col = (head < G ? hk * G + head : head == G ? a.hq + hk : a.hq + a.hkv + hk) * HD + j;
      const RotaryPlanes x = raw_planes(a.raw, i, col, half, j, head <= G);
      if (head < G) { *(f32x4_t *)&qs[head][j] = x.a; *(f32x4_t *)&qs[head][j + half] = x.b; continue; }
      const uint2 x0 = pack4(x.a), x1 = pack4(x.b);
      T *const o = own + (head - G) * HD + j, *const c = cache[head - G] + at + j;
      *(uint2 *)o = x0; *(uint2 *)(o + half) = x1;
      if (store) { *(uint2 *)c = x0; *(uint2 *)(c + half) = x1; }
    }
  } else {
    const float *qrow = (const float *)a.q + ((size_t)i * a.hq + (size_t)hk * G) * HD;   // queries are fp32
    for (int e = lane; e < G * HD; e += 64) qs[e / HD][e % HD] = qrow[e];
  }
  wave_lds_sync();
  if (mine) {
#pragma unroll
    for (int dc = 0; dc < QC; dc++) {
      kc[dc] = *(const u32x4_t *)(own + qt * QD + dc * EPL);
      vc[dc] = *(const u32x4_t *)(own + HD + qt * QD + dc * EPL);
    }
  }
  float s[G];
#pragma unroll
  for (int gh = 0; gh < G; gh++) s[gh] = 0.f;
#pragma unroll
  for (int dc = 0; dc < QC; dc++) {
    float kf[EPL];
    Chunk<T>::unpack(kc[dc], kf);
#pragma unroll
    for (int gh = 0; gh < G; gh++)
#pragma unroll
      for (int e = 0; e < EPL; e++) s[gh] = fmaf(qs[gh][qt * QD + dc * EPL + e], kf[e], s[gh]);
  }
#pragma unroll
  for (int dc = 0; dc < QC; dc++) *(u32x4_t *)(vs + kk * VROW + qt * QD * (int)sizeof(T) + dc * 16) = vc[dc];
  float m_run[G], l_run[G], pk[G];
#pragma unroll
  for (int gh = 0; gh < G; gh++) {
    float t = s[gh];
    t += dpp_f32<0xB1>(t);                           // quad sum, fixed order: quad_perm [1,0,3,2], [2,3,0,1]
    t += dpp_f32<0x4E>(t);
    const float sc = valid ? t * a.scale : -INFINITY;
    m_run[gh] = wave_max(sc);                        // at least key p itself is valid
    pk[gh] = valid ? exp2_(sc - m_run[gh]) : 0.f;
    l_run[gh] = wave_sum(qt == 0 ? pk[gh] : 0.f);
  }
  wave_lds_sync();                                   // value rows staged
  float o[G][DPL];
#pragma unroll
  for (int gh = 0; gh < G; gh++)
#pragma unroll
    for (int dd = 0; dd < DPL; dd++) o[gh][dd] = 0.f;
  // Lanes of keys past p hold weight 0 and a finite value row (a copy of the row's own), so all 16 rows can be summed.
  const unsigned char *vcol = vs + lane * DPL * (int)sizeof(T);
#pragma unroll
  for (int k0 = 0; k0 < kTailKeys; k0 += 8) {
    float vv[8][DPL];
#pragma unroll
    for (int u = 0; u < 8; u++)
#pragma unroll
      for (int dd = 0; dd < DPL; dd++) vv[u][dd] = to_f32(*(const T *)(vcol + (k0 + u) * VROW + dd * (int)sizeof(T)));
#pragma unroll
    for (int u = 0; u < 8; u++)
#pragma unroll
      for (int gh = 0; gh < G; gh++) {
        const float w = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(pk[gh]), (k0 + u) * 4));
#pragma unroll
        for (int dd = 0; dd < DPL; dd++) o[gh][dd] = fmaf(w, vv[u][dd], o[gh][dd]);
      }
  }
  if (!store) return;
#pragma unroll
  for (int gh = 0; gh < G; gh++) {
    float *dst = a.part + (((size_t)i * a.hq + hk * G + gh) * a.max_parts + a.max_parts - 1) * (HD + 2);
    if (lane == 0) { dst[0] = m_run[gh]; dst[1] = l_run[gh]; }
#pragma unroll
    for (int dd = 0; dd < DPL; dd++) dst[2 + lane * DPL + dd] = o[gh][dd];
  }
}

// grid (rows, kv heads, parts); one wavefront per workgroup.
template <typename T, int HD, int G>
__global__ __launch_bounds__(64) void attn_part_kernel(AttnArgs a) {
  __shared__ __attribute__((aligned(16))) float qs[G][HD];
  __shared__ __attribute__((aligned(16))) unsigned char vs[64 * PartLds<T>::vrow(HD)];
  const int lane = threadIdx.x;
  float *const dst0 = a.part + (((size_t)blockIdx.x * a.hq + blockIdx.y * G) * a.max_parts + blockIdx.z) * (HD + 2);
  attn_part_body<T, HD, G, false>(a, blockIdx.x, blockIdx.y, blockIdx.z, lane, qs, vs, [&](int gh, float m, float l, const float (&o)[HD / 64]) __attribute__((always_inline)) {
    float *dst = dst0 + (size_t)gh * a.max_parts * (HD + 2);
    if (lane == 0) { dst[0] = m; dst[1] = l; }
#pragma unroll
    for (int dd = 0; dd < HD / 64; dd++) dst[2 + lane * (HD / 64) + dd] = o[dd];
  });
}

// fp32 storage, short contexts: grid (rows, kv heads), a wavefront per part (up to kRowParts), the parts merged in the LDS as attn_combine_kernel merges them,
// bit for bit.  One launch instead of two and no partial outputs in memory: request of the small fp32 model 4.76 -> 4.63 ms (bound: latency; the launch saved is 1.2 us
// of each layer and draft pass, the partial outputs' way as much again).
constexpr int kRowParts = 4;
template <int HD, int G> constexpr int row_wave_bytes() { return G * HD * 4 + 64 * PartLds<float>::vrow(HD); }
template <int HD, int G>
__global__ __launch_bounds__(kRowParts * 64, 1) void attn_row_kernel(AttnArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char row_lds[];
  __shared__ float pm[kRowParts][G], pl[kRowParts][G];
  const int i = blockIdx.x, hk = blockIdx.y, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n_parts = attn_parts_covering((a.base_ptr ? *a.base_ptr : a.base) + a.depth[i] + 1);
  unsigned char *const mine = row_lds + wave * row_wave_bytes<HD, G>();
  attn_part_body<float, HD, G, HD == 64>(a, i, hk, wave, lane, (float (*)[HD])mine, mine + G * HD * 4, [&](int gh, float m, float l, const float (&o)[HD / 64]) __attribute__((always_inline)) {
    if (lane == 0) { pm[wave][gh] = m; pl[wave][gh] = l; }
#pragma unroll
    for (int dd = 0; dd < HD / 64; dd++) ((float *)mine)[gh * HD + lane * (HD / 64) + dd] = o[dd];   // (the query's place)
  });
  __syncthreads();
  for (int e = threadIdx.x; e < G * HD; e += blockDim.x) {
    RowMerge row;
    float o = 0.f;
    for (int t = 0; t < n_parts; t++) {
      float w;
      const float turn = row.step(pm[t][e / HD], pl[t][e / HD], w);
      o = fmaf(*(const float *)(row_lds + t * row_wave_bytes<HD, G>() + e * 4), w, o * turn);
    }
    ((float *)a.out)[((size_t)i * a.hq + (size_t)hk * G) * HD + e] = o / row.l;
  }
}

// grid (rows, hq); block HD threads.  Merges the row's parts in ascending order (RowMerge); in hybrid mode these are
// the bulk parts followed by the tail (kept in the last slot).  The (reference, sum) pairs of up to kCombineChunk
// parts are fetched by one thread each, so that the per-dim pass issues independent, coalesced loads.
constexpr int kCombineChunk = 64;
constexpr int kCombineFew = 8;         // up to this many parts a thread keeps everything in registers
template <typename T, int HD>
__global__ __launch_bounds__(HD) void attn_combine_kernel(AttnArgs a) {
  __shared__ float pm[kCombineChunk], pl[kCombineChunk];
  const int i = blockIdx.x, h = blockIdx.y, d = threadIdx.x;
  const int p = (a.base_ptr ? *a.base_ptr : a.base) + a.depth[i];
  const int n_front = attn_parts_covering(a.tail_only ? bulk_end(p) : p + 1);
  const int n_parts = n_front + (a.tail_only ? 1 : 0);
  const float *src = a.part + ((size_t)i * a.hq + h) * a.max_parts * (HD + 2);
  auto slot = [&](int t) { return (size_t)(t < n_front ? t : a.max_parts - 1) * (HD + 2); };
  if (n_parts <= kCombineFew) {
    // Few parts (short contexts): every value is requested up front (clamped to a valid part; absent ones are not used),
    // then the same arithmetic as below runs out of registers: one memory round trip instead of three.
    float pm_[kCombineFew], pl_[kCombineFew], pv_[kCombineFew];
#pragma unroll
    for (int t = 0; t < kCombineFew; t++) {
      const float *sp = src + slot(t < n_parts ? t : 0);
      pm_[t] = sp[0]; pl_[t] = sp[1]; pv_[t] = sp[2 + d];
    }
    RowMerge row;
    float o = 0.f;
#pragma unroll
    for (int t = 0; t < kCombineFew; t++)
      if (t < n_parts) {
        float w;
        const float turn = row.step(pm_[t], pl_[t], w);
        o = fmaf(pv_[t], w, o * turn);
      }
    ((T *)a.out)[((size_t)i * a.hq + h) * HD + d] = from_f32<T>(o / row.l);
    return;
  }
  // chunks of parts: the (reference, sum) pairs through the LDS, the outputs of four parts in flight; every thread steps through all of them
  RowMerge row;
  float o = 0.f;
  for (int t0 = 0; t0 < n_parts; t0 += kCombineChunk) {
    const int nt = min(kCombineChunk, n_parts - t0);
    if (t0 > 0) __syncthreads();
    if (d < nt) { const float *sp = src + slot(t0 + d); pm[d] = sp[0]; pl[d] = sp[1]; }
    __syncthreads();
    auto add = [&](int t, float v) __attribute__((always_inline)) {
      float w;
      const float turn = row.step(pm[t], pl[t], w);
      o = fmaf(v, w, o * turn);
    };
    int t = 0;
    for (; t + 4 <= nt; t += 4) {
      const float v0 = src[slot(t0 + t) + 2 + d], v1 = src[slot(t0 + t + 1) + 2 + d];
      const float v2 = src[slot(t0 + t + 2) + 2 + d], v3 = src[slot(t0 + t + 3) + 2 + d];
      add(t, v0); add(t + 1, v1); add(t + 2, v2); add(t + 3, v3);
    }
    for (; t < nt; t++) add(t, src[slot(t0 + t) + 2 + d]);
  }
  ((T *)a.out)[((size_t)i * a.hq + h) * HD + d] = from_f32<T>(o / row.l);
}

// ---- matrix-core path for the bulk region (bf16 storage) -----------------------------------
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;


// x = hi + lo with hi, lo bf16: the pair keeps ~16 mantissa bits of an fp32 value.
__device__ __forceinline__ void split8(const float (&x)[8], u32x4_t &hi, u32x4_t &lo) {
  uint32_t h[4], l[4];
#pragma unroll
  for (int e = 0; e < 4; e++) {
    h[e] = pack_bf16x2(x[2 * e], x[2 * e + 1]);
    l[e] = pack_bf16x2(x[2 * e] - __uint_as_float(h[e] << 16), x[2 * e + 1] - __uint_as_float(h[e] & 0xFFFF0000u));
  }
  hi = u32x4_t{h[0], h[1], h[2], h[3]};
  lo = u32x4_t{l[0], l[1], l[2], l[3]};
}
__device__ __forceinline__ f32x16_t mfma_bf16(const u32x4_t &a, const u32x4_t &b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// four floats at a 4-byte aligned address in one store
__device__ __forceinline__ void store4_any(float *p, float a, float b, float c, float d) {
  typedef __attribute__((ext_vector_type(4), aligned(4))) float f4_t;
  *(f4_t *)p = f4_t{a, b, c, d};
}

// Sum over the lanes l and l ^ 32, in both (max_halves)
__device__ __forceinline__ float sum_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// The running softmax of a part over a block of 32 keys: s[v] = q . k (masked keys -inf), a lane and lane ^ 32 share a query.  The reference m moves
// only when the block's maximum exceeds it by more than kRefSlack, as in RowMerge: the output registers (times `turn`) are seldom touched.
struct PartSoftmax {
  float m = -INFINITY, l = 0.f;
  // turn: what the part's outputs are to be multiplied by (1 unless some query of the wavefront moves); p[v]: the keys' weights
  __device__ __forceinline__ bool block(const f32x16_t &s, float scale, float &turn, float (&p)[16]) {
    float mb = -INFINITY;
#pragma unroll
    for (int v = 0; v < 16; v++) mb = fmaxf(mb, s[v]);
    mb = max_halves(mb) * scale;                              // (the scale is positive and rounding keeps order)
    const bool move = mb > m + kRefSlack;                      // also the first key
    const bool any = __any(move);
    turn = 1.f;
    if (any) {
      const float m_new = move ? mb : m;
      turn = move ? exp2_(m - m_new) : 1.f;
      m = m_new;
    }
    const float m_use = m == -INFINITY ? 0.f : m;              // nothing seen yet: every term is 0
    float ls = 0.f;
#pragma unroll
    for (int v = 0; v < 16; v++) { p[v] = exp2_(fmaf(s[v], scale, -m_use)); ls += p[v]; }
    l = fmaf(l, turn, sum_halves(ls));
    return any;
  }
};

// One launch covers both regions of the hybrid path.  Workgroups [0, n_bulk) (n_bulk = bulk_parts * kv heads
// * q_groups, part fastest) run the matrix-core bulk: NW waves, wave w owns 32 "query rows" (row i, head gh
// of the kv group), r = (qgroup*NW + w)*32 + lane%32, i = r / G, gh = r % G.  The remaining workgroups run
// the vector tail, one (row, kv head) item per wavefront on the first kTailWaves wavefronts, and leave it in
// the last part slot.  The two kinds of work are independent; attn_combine_kernel merges them afterwards.
#ifndef SPEC_ATTN_RING
#define SPEC_ATTN_RING 1
#endif
constexpr int kBulkRing = SPEC_ATTN_RING;   // register sets for K/V blocks in flight per bulk workgroup
template <int NW> struct TailWaves { static constexpr int value = NW < 4 ? NW : 4; };
// RAW: queries, keys and values come from the QKV projection's partial sums: every bulk workgroup forms its queries, a tail wavefront its row's query, key and
// value.  The launch for that, 4.7 us ahead of this one, was mostly the way from launch to launch: 7B, one row at 90 keys 4.7 + 6.7 -> 7.0 us, a draft
// pass of ten rows at 530 4.8 + 8.4 -> 9.1, 8B, ten rows (40 queries to a key) at 4100 4.8 + 13.6 -> 16.0, four at 1340 4.9 + 12.2 -> 13.4.
template <int HD, int G, int NW, bool RAW = false>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_hybrid_kernel(AttnArgs a) {
  constexpr int DB = HD / 32;                 // 32-dim blocks of the output
  constexpr int KK = HD / 16;                 // MFMA steps of q.k
  constexpr int KSTR = HD * 2 + 16;           // LDS bytes per key row (+16: conflict-free b128 reads)
  constexpr int NT = NW * 64;
  constexpr int PIECES = (32 * HD * 2 / 16 + NT - 1) / NT;   // 16-byte pieces of one K (or V) block per thread
  constexpr int kTailWaves = TailWaves<NW>::value;
  constexpr int kTailQ = G * HD * 4;                                         // a tail wavefront's query area
  constexpr int kTailVs = kTailQ + kTailKeys * PartLds<bf16_t>::vrow(HD);    // ... plus its staged value rows
  constexpr int kTailWave = kTailVs + (RAW ? 2 * HD * 2 : 0);                // ... plus the row's own key and value
  constexpr int kBulkBuf = 32 * KSTR + 32 * HD * 2;                          // one staged K block + V block
  constexpr int kBulkLds = 2 * kBulkBuf;                                     // double-buffered
  constexpr int kLds = kBulkLds > kTailWaves * kTailWave ? kBulkLds : kTailWaves * kTailWave;
  __shared__ __attribute__((aligned(16))) unsigned char lds[kLds];
  static_assert(!RAW || kRawQueries * HD * 4 <= kLds, "the queries lie where the keys and values will");

  const int n_bulk = a.bulk_parts * a.hkv * a.q_groups;
  if ((int)blockIdx.x >= n_bulk) {
    const int w = threadIdx.x >> 6;
    if (w >= kTailWaves) return;
    int item = ((int)blockIdx.x - n_bulk) * kTailWaves + w;
    const bool active = item < a.rows * a.hkv;
    if (!active) item = a.rows * a.hkv - 1;               // valid addresses; result discarded
    unsigned char *mine = lds + w * kTailWave;
    attn_tail_body<bf16_t, HD, G, RAW>(a, item / a.hkv, item % a.hkv, threadIdx.x & 63, (float (*)[HD])mine, mine + kTailQ, active, (bf16_t *)(mine + kTailVs));
    return;
  }
  const int part = (int)blockIdx.x % a.bulk_parts, hk = ((int)blockIdx.x / a.bulk_parts) % a.hkv;
  const int qgroup = (int)blockIdx.x / (a.bulk_parts * a.hkv);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, c = lane & 31, g = lane >> 5;
  // With a device-resident base (graph replay) the grid is sized for the longest context and the
  // blocks that exist are derived here; otherwise the host has computed them.
  const int base = a.base_ptr ? *a.base_ptr : a.base;
  // keys [0, key_lim) are the union of the rows' bulk regions: all of them exist and are initialised
  const int key_lim = a.base_ptr ? min(a.bulk_keys, bulk_end(base + kMaxDepth)) : a.bulk_keys;
  const int n_blocks = (key_lim + 31) / 32;
  const int b_lo = attn_part_begin(part) / 32;
  const int b_hi = min(attn_part_begin(part + 1) / 32, n_blocks);
  if (b_lo >= b_hi) return;

  const int r = (qgroup * NW + wave) * 32 + c;
  const bool valid_q = r < a.rows * G;
  const int i = valid_q ? r / G : 0, gh = valid_q ? r % G : 0;
  const int k_end = valid_q ? bulk_end(base + a.depth[i]) : 0;               // keys [0, k_end) belong to this row's bulk

  const size_t row_stride = (size_t)a.hkv * HD;              // elements between consecutive cache slots
  const bf16_t *kg = (const bf16_t *)a.kcache + (size_t)hk * HD;
  const bf16_t *vg = (const bf16_t *)a.vcache + (size_t)hk * HD;
  constexpr int PPR = HD * 2 / 16;                           // pieces per key row
  // The global loads of a block land in one of R register sets, so that R blocks are in flight.  Measured on
  // MI355X, more than one set does not pay: the arithmetic of a block, not the wait for its loads, is what a
  // workgroup spends its time on.
  constexpr int R = kBulkRing;
  u32x4_t kreg[R][PIECES], vreg[R][PIECES];
  auto prefetch = [&](auto set_tag, int b) {
    constexpr int SET = decltype(set_tag)::value;
#pragma unroll
    for (int e = 0; e < PIECES; e++) {
      const int q = tid + e * NT;
      const int key = (q / PPR) & 31, piece = q % PPR;       // (& 31: threads past the block re-read a valid key)
      // The last block may reach past key_lim; those keys are masked for every row, so they are read from
      // key key_lim - 1 instead (initialised, inside the cache; key_lim >= 1 for every block that runs).
      const size_t off = (size_t)min(b * 32 + key, key_lim - 1) * row_stride + piece * 8;
      kreg[SET][e] = *(const u32x4_t *)(kg + off);
      vreg[SET][e] = *(const u32x4_t *)(vg + off);
    }
  };
  // A wavefront whose 32 query rows all lie past the last row only helps to load and stage the blocks.
  const bool computes = __builtin_amdgcn_readfirstlane((qgroup * NW + wave) * 32 < a.rows * G ? 1 : 0) != 0;
  u32x4_t qhi[KK], qlo[KK];                                  // query fragments: step kk covers dims kk*16 + g*8 .. +8
  f32x16_t o[DB];
#pragma unroll
  for (int db = 0; db < DB; db++)
#pragma unroll
    for (int v = 0; v < 16; v++) o[db][v] = 0.f;
  PartSoftmax run_;
  const int vat = value_lane<HD>(lane);
  int k_low = k_end;                                         // the least over the wavefront's rows
#pragma unroll
  for (int x = 1; x < 32; x <<= 1) k_low = min(k_low, __shfl_xor(k_low, x, 64));
  k_low = __builtin_amdgcn_readfirstlane(k_low);

  auto stage = [&](auto set_tag, int buf) {
    constexpr int SET = decltype(set_tag)::value;
    unsigned char *k_lds = lds + buf * kBulkBuf, *v_lds = k_lds + 32 * KSTR;
#pragma unroll
    for (int e = 0; e < PIECES; e++) {
      const int q = tid + e * NT;
      if (q < 32 * PPR) {
        const int key = q / PPR, piece = q % PPR;
        *(u32x4_t *)(k_lds + key * KSTR + piece * 16) = kreg[SET][e];
        *(u32x4_t *)(v_lds + value_piece<HD>(key, piece)) = vreg[SET][e];
      }
    }
  };

  // One part = NB blocks, b_lo .. b_lo + NB - 1, as straight-line code: every load and every wait for a load
  // is unconditional, so the compiler counts outstanding loads exactly and a block waits for its own set only.
  // Blocks at or past b_hi (a part cut short by the end of the keys) are loaded from clamped addresses, staged
  // and skipped by the arithmetic.  K/V blocks alternate between two LDS buffers: block j+1 is staged between the
  // two matrix-core phases of block j and its register set is refilled right away with block j+1+R; one barrier
  // per block.
  auto run = [&](auto nb_tag) {
    constexpr int NB = decltype(nb_tag)::value;
    static_assert(NB >= 1 && NB <= 16, "a part is unrolled block by block");
    if constexpr (RAW) {
      constexpr int per_head = HD / 8;
      for (int e = tid; e < a.rows * G * per_head; e += NT) { // (rows * G <= kRawQueries)
        const int query = e / per_head, j = e % per_head * 4;
        const RotaryPlanes x = raw_planes(a.raw, query / G, (hk * G + query % G) * HD + j, HD / 2, j, true);
        *(f32x4_t *)((float *)lds + query * HD + j) = x.a;
        *(f32x4_t *)((float *)lds + query * HD + j + HD / 2) = x.b;
      }
    }
    unrolled<(R < NB ? R : NB)>([&](auto t_tag) { prefetch(t_tag, b_lo + decltype(t_tag)::value); });
    if constexpr (RAW) __syncthreads();
    {
      const float *qrow = RAW ? (const float *)lds + (i * G + gh) * HD : (const float *)a.q + ((size_t)i * a.hq + (size_t)hk * G + gh) * HD;
#pragma unroll
      for (int kk = 0; kk < KK; kk++) {
        float x[8];
        const float4 x0 = *(const float4 *)(qrow + kk * 16 + g * 8), x1 = *(const float4 *)(qrow + kk * 16 + g * 8 + 4);
        x[0] = x0.x; x[1] = x0.y; x[2] = x0.z; x[3] = x0.w; x[4] = x1.x; x[5] = x1.y; x[6] = x1.z; x[7] = x1.w;
        split8(x, qhi[kk], qlo[kk]);
      }
    }
    if constexpr (RAW) __syncthreads();
    stage(std::integral_constant<int, 0>{}, 0);
    __syncthreads();
    if constexpr (R < NB) prefetch(std::integral_constant<int, 0>{}, b_lo + R);
    unrolled<NB>([&](auto j_tag) {
      constexpr int j = decltype(j_tag)::value, cur = j & 1;
      const int b = b_lo + j;
      const bool live = computes && b < b_hi;                // same for all lanes of a wavefront
      const unsigned char *k_lds = lds + cur * kBulkBuf, *v_lds = k_lds + 32 * KSTR;
      float pv[16];
      if (live) {
        f32x16_t s;
#pragma unroll
        for (int v = 0; v < 16; v++) s[v] = 0.f;
#pragma unroll
        for (int kk = 0; kk < KK; kk++) {
          const u32x4_t kf = *(const u32x4_t *)(k_lds + c * KSTR + kk * 32 + g * 16);
          s = mfma_bf16(kf, qhi[kk], s);
          s = mfma_bf16(kf, qlo[kk], s);
        }
        // s[v] = q . k for key 8*(v/4) + 4*g + v%4 of the block and query row c
        // keys at or past k_end are masked: they add exact zeros, so a row's result does not depend on them
        const int key0 = b * 32 + 4 * g;
        if (b * 32 + 32 > k_low) {                            // some row of the wavefront ends inside the block
#pragma unroll
          for (int v = 0; v < 16; v++)
            if (key0 + 8 * (v >> 2) + (v & 3) >= k_end) s[v] = -INFINITY;
        }
        float turn;
        if (run_.block(s, a.scale, turn, pv)) {
#pragma unroll
          for (int db = 0; db < DB; db++)
#pragma unroll
            for (int v = 0; v < 16; v++) o[db][v] *= turn;
        }
      }
      if constexpr (j + 1 < NB) {
        constexpr int NEXT = (j + 1) % R;
        stage(std::integral_constant<int, NEXT>{}, cur ^ 1);   // every wave left that buffer at the last barrier
        if constexpr (j + 1 + R < NB) prefetch(std::integral_constant<int, NEXT>{}, b + 1 + R);
      }
      if (live) {
        // O^T += V^T P^T over two 16-key steps; step u uses the lane's own values v = 8u .. 8u+7,
        // i.e. keys 16u + 8*(e/4) + 4g + e%4, and V^T supplies the same keys per dim.
#pragma unroll
        for (int u = 0; u < 2; u++) {
          float x[8];
#pragma unroll
          for (int e = 0; e < 8; e++) x[e] = pv[8 * u + e];
          u32x4_t phi, plo;
          split8(x, phi, plo);
#pragma unroll
          for (int db = 0; db < DB; db++) {
            const u32x4_t vf = value_fragment<HD>(v_lds, vat, db, 16 * u);
            o[db] = mfma_bf16(vf, phi, o[db]);
            o[db] = mfma_bf16(vf, plo, o[db]);
          }
        }
      }
      if constexpr (j + 1 < NB) __syncthreads();             // block j+1 staged; everyone is done with block j
    });
  };
  if (part < kAttnNear / kAttnPart) run(std::integral_constant<int, kAttnPart / 32>{});
  else run(std::integral_constant<int, kAttnFarPart / 32>{});
  if (!valid_q) return;
  float *dst = a.part + (((size_t)i * a.hq + hk * G + gh) * a.max_parts + part) * (HD + 2);
  if (g == 0) { dst[0] = run_.m; dst[1] = run_.l; }
#pragma unroll
  for (int db = 0; db < DB; db++)
#pragma unroll
    for (int v = 0; v < 16; v += 4) store4_any(dst + 2 + db * 32 + 2 * v + 4 * g, o[db][v], o[db][v + 1], o[db][v + 2], o[db][v + 3]);
}

template <int HD, int G, int NW>
static hipError_t launch_hybrid(AttnArgs a, int q_groups, hipStream_t st) {
  a.q_groups = q_groups;
  const int n_tail = (a.rows * a.hkv + TailWaves<NW>::value - 1) / TailWaves<NW>::value;
  const dim3 grid(a.bulk_parts * a.hkv * q_groups + n_tail), threads(NW * 64);
  if constexpr (NW == 4) {
    if (a.raw.qkv != nullptr) {
      hipLaunchKernelGGL((attn_hybrid_kernel<HD, G, NW, true>), grid, threads, 0, st, a);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((attn_hybrid_kernel<HD, G, NW>), grid, threads, 0, st, a);
  return hipGetLastError();
}

// ---- many rows of a causal chain (prefill), bf16 storage ---------------------------------------
// The same arithmetic as the hybrid path and its merge, bit for bit, without partial outputs of the bulk in memory: with hundreds of
// rows a row's keys need no split over workgroups (512 rows at 4096 keys, 32 heads: 170 MB of partials per layer).  The tails run
// first (attn_tail_kernel: one wavefront per row and kv head, fp32) and leave their partial; then one workgroup of WAVES
// wavefronts takes WAVES * 32 consecutive rows of one query head and walks their bulk keys: the running softmax of every part as the hybrid
// path does it (32 keys at a time, from nothing per part), and each finished part goes into the row's sums as the merge does it (RowMerge
// needs no maximum ahead of time, so that one walk is enough; a merge weighted by the row's maximum took a walk over all keys for that alone).
// Two sets of output registers (part and row) leave no room for both query terms at head dim 128: the low one is read from the LDS.
// K and V blocks are double-buffered there, the loads of a block run two blocks ahead.  Rows may stand at any positions
// (depth); a block past a wavefront's last bulk key is skipped (it would add exact zeros).
// Bound: from one full chip of workgroups on the matrix cores, below that the serial chain of a block.
// Measured (MI355X, us per call with the tails; in two walks, references moving at every new maximum, before): 512 rows, 32 heads 58 -> 48; 1024 rows,
// 64 heads on 8 kv heads 134 -> 110; 1333 rows, 32 on 8 115 -> 87; 2048 rows 177 -> 130, at 2048 keys before them 355 -> 251.
template <int HD, int WAVES> struct ChainLds {
  static constexpr int kKeys = HD == 128 ? 32 : 64;   // keys per staged block: what the registers beside queries and outputs leave
  static constexpr int kstr = HD * 2 + 16;            // bytes per staged key row (+16: conflict-free b128 reads)
  static constexpr int buf = kKeys * kstr + kKeys * HD * 2;
  static constexpr bool kQueryLds = HD == 128;
  static constexpr int total = 2 * buf + (kQueryLds ? WAVES * (HD / 16) * 1024 : 0);
};
template <int HD, int WAVES>
__global__ __launch_bounds__(WAVES * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_chain_kernel(AttnArgs a) {
  using L = ChainLds<HD, WAVES>;
  constexpr int NT = WAVES * 64, KEYS = L::kKeys, KT = KEYS / 32;
  constexpr int DB = HD / 32, KK = HD / 16, PPR = HD * 2 / 16;
  constexpr int KP = KEYS * PPR / NT;
  static_assert(KEYS * PPR % NT == 0, "staging split");
  static_assert(kAttnPart % KEYS == 0 && kAttnNear % KEYS == 0 && kAttnFarPart % KEYS == 0, "a part ends with a staged block");
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  __shared__ int wave_hi[WAVES];

  // Workgroup -> (head, row tile): last tile (the longest) first; with a multiple of eight kv heads all workgroups of a kv head
  // run on one XCD (ids 8 apart) and share its keys and values through that L2.
  const int G = a.hq / a.hkv, n_qt = (a.rows + WAVES * 32 - 1) / (WAVES * 32);
  const bool affine = (a.hkv & 7) == 0;
  const int lists = affine ? 8 : 1, heads = a.hq / lists;     // heads per list
  const int id = (int)blockIdx.x / lists, list = (int)blockIdx.x % lists;
  const int qt = n_qt - 1 - id / heads, hl = id % heads;
  const int hk = (hl / G) * lists + list, h = hk * G + hl % G;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, c = lane & 31, g = lane >> 5;
  const int i = (qt * WAVES + wave) * 32 + c;                 // row of this lane
  const bool valid = i < a.rows;
  const int base = a.base_ptr ? *a.base_ptr : a.base;
  const int k_end = valid ? bulk_end(base + a.depth[i]) : 0;  // keys [0, k_end) belong to this row's bulk
  int lo = valid ? k_end : 0x7FFFFFFF, hi = k_end;            // over the wavefront's rows
#pragma unroll
  for (int o = 1; o < 32; o <<= 1) { lo = min(lo, __shfl_xor(lo, o, 64)); hi = max(hi, __shfl_xor(hi, o, 64)); }
  lo = __builtin_amdgcn_readfirstlane(lo); hi = __builtin_amdgcn_readfirstlane(hi);
  if (lane == 0) wave_hi[wave] = hi;
  __syncthreads();
  int k_wg = wave_hi[0];                                      // the workgroup's bulk keys are [0, k_wg)
#pragma unroll
  for (int w = 1; w < WAVES; w++) k_wg = max(k_wg, wave_hi[w]);
  k_wg = __builtin_amdgcn_readfirstlane(k_wg);

  const size_t kv_stride = (size_t)a.hkv * HD;
  const bf16_t *kg = (const bf16_t *)a.kcache + (size_t)hk * HD, *vg = (const bf16_t *)a.vcache + (size_t)hk * HD;
  // keys past the workgroup's last are read from it and masked
  auto piece_of = [&](const bf16_t *p, int key, int piece) { return *(const u32x4_t *)(p + (size_t)min(key, k_wg - 1) * kv_stride + piece * 8); };

  u32x4_t qhi[KK], qlo[KK];                                   // step kk covers dims kk*16 + g*8 .. +8 of the lane's query
  {
    const float *qrow = (const float *)a.q + ((size_t)(valid ? i : a.rows - 1) * a.hq + h) * HD;
#pragma unroll
    for (int kk = 0; kk < KK; kk++) {
      float x[8];
      const float4 x0 = *(const float4 *)(qrow + kk * 16 + g * 8), x1 = *(const float4 *)(qrow + kk * 16 + g * 8 + 4);
      x[0] = x0.x; x[1] = x0.y; x[2] = x0.z; x[3] = x0.w; x[4] = x1.x; x[5] = x1.y; x[6] = x1.z; x[7] = x1.w;
      split8(x, qhi[kk], qlo[kk]);
    }
  }
  unsigned char *q_lds = lds + 2 * L::buf + wave * (KK * 1024) + lane * 16;
  if constexpr (L::kQueryLds) {
#pragma unroll
    for (int kk = 0; kk < KK; kk++) *(u32x4_t *)(q_lds + kk * 1024) = qlo[kk];
  }
  const float *tail = a.part + (((size_t)(valid ? i : a.rows - 1) * a.hq + h) * a.max_parts + a.max_parts - 1) * (HD + 2);

  f32x16_t o[DB], row[DB];                                    // output of the part under way, and of the row
#pragma unroll
  for (int db = 0; db < DB; db++)
#pragma unroll
    for (int v = 0; v < 16; v++) o[db][v] = row[db][v] = 0.f;
  PartSoftmax part;
  RowMerge merge;
  auto turn_row = [&](float turn) __attribute__((always_inline)) {
    if (__any(turn != 1.f)) {
#pragma unroll
      for (int db = 0; db < DB; db++)
#pragma unroll
        for (int v = 0; v < 16; v++) row[db][v] *= turn;
    }
  };

  if (k_wg > 0) {
    u32x4_t kreg[KP], vreg[KP];
    const int nb = (k_wg + KEYS - 1) / KEYS;
    auto prefetch = [&](int blk) {
#pragma unroll
      for (int e = 0; e < KP; e++) {
        const int q = tid + e * NT;
        kreg[e] = piece_of(kg, blk * KEYS + q / PPR, q % PPR);
        vreg[e] = piece_of(vg, blk * KEYS + q / PPR, q % PPR);
      }
    };
    auto stage = [&](int b) {
      unsigned char *k_lds = lds + b * L::buf, *v_lds = k_lds + KEYS * L::kstr;
#pragma unroll
      for (int e = 0; e < KP; e++) {
        const int q = tid + e * NT;
        *(u32x4_t *)(k_lds + (q / PPR) * L::kstr + (q % PPR) * 16) = kreg[e];
        *(u32x4_t *)(v_lds + value_piece<HD>(q / PPR, q % PPR)) = vreg[e];
      }
    };
    const int vat = value_lane<HD>(lane);
    prefetch(0);
    stage(0);
    __syncthreads();
    if (nb > 1) prefetch(1);
    int part_lo = 0;                                          // first key of the part under way
    for (int blk = 0; blk < nb; blk++) {
      const unsigned char *k_lds = lds + (blk & 1) * L::buf, *v_lds = k_lds + KEYS * L::kstr;
      if (blk + 1 < nb) {
        stage((blk + 1) & 1);
        if (blk + 2 < nb) prefetch(blk + 2);
      }
      if (blk * KEYS < hi) {
#pragma unroll
        for (int kt = 0; kt < KT; kt++) {
          f32x16_t s;
#pragma unroll
          for (int v = 0; v < 16; v++) s[v] = 0.f;
#pragma unroll
          for (int kk = 0; kk < KK; kk++) {
            const u32x4_t kf = *(const u32x4_t *)(k_lds + (kt * 32 + c) * L::kstr + kk * 32 + g * 16);
            u32x4_t ql;
            if constexpr (L::kQueryLds) ql = *(const u32x4_t *)(q_lds + kk * 1024);
            else ql = qlo[kk];
            s = mfma_bf16(kf, qhi[kk], s);
            s = mfma_bf16(kf, ql, s);
          }
          const int b0 = blk * KEYS + kt * 32;
          if (b0 + 32 > lo) {                                 // some row ends inside the block
            const int key0 = b0 + 4 * g;
#pragma unroll
            for (int v = 0; v < 16; v++)
              if (key0 + 8 * (v >> 2) + (v & 3) >= k_end) s[v] = -INFINITY;
          }
          float turn, pv[16];
          if (part.block(s, a.scale, turn, pv)) {
#pragma unroll
            for (int db = 0; db < DB; db++)
#pragma unroll
              for (int v = 0; v < 16; v++) o[db][v] *= turn;
          }
#pragma unroll
          for (int u = 0; u < 2; u++) {                       // 16 keys: the lane's own values v = 8u .. 8u+7
            float x[8];
#pragma unroll
            for (int e = 0; e < 8; e++) x[e] = pv[8 * u + e];
            u32x4_t phi, plo;
            split8(x, phi, plo);
#pragma unroll
            for (int db = 0; db < DB; db++) {
              const u32x4_t vf = value_fragment<HD>(v_lds, vat, db, 32 * kt + 16 * u);
              o[db] = mfma_bf16(vf, phi, o[db]);
              o[db] = mfma_bf16(vf, plo, o[db]);
            }
          }
        }
        const int done = (blk + 1) * KEYS;
        if (done >= hi || (done <= kAttnNear ? done % kAttnPart : (done - kAttnNear) % kAttnFarPart) == 0) {
          if (part_lo < k_end) {                              // this row has keys in the part
            float w;
            turn_row(merge.step(part.m, part.l, w));
#pragma unroll
            for (int db = 0; db < DB; db++)
#pragma unroll
              for (int v = 0; v < 16; v++) row[db][v] = fmaf(o[db][v], w, row[db][v]);
          }
#pragma unroll
          for (int db = 0; db < DB; db++)
#pragma unroll
            for (int v = 0; v < 16; v++) o[db][v] = 0.f;
          part = PartSoftmax{};
          part_lo = done;
        }
      }
      __syncthreads();                                        // block blk+1 staged; everyone is done with block blk
    }
  }
  float w;
  turn_row(merge.step(tail[0], tail[1], w));
  if (!valid) return;
  bf16_t *orow = (bf16_t *)a.out + ((size_t)i * a.hq + h) * HD;
#pragma unroll
  for (int db = 0; db < DB; db++)
#pragma unroll
    for (int q4 = 0; q4 < 4; q4++) {
      const int d0 = db * 32 + 8 * q4 + 4 * g;
      const float2 t0 = *(const float2 *)(tail + 2 + d0), t1 = *(const float2 *)(tail + 2 + d0 + 2);
      const float t[4] = {t0.x, t0.y, t1.x, t1.y};
      float y[4];
#pragma unroll
      for (int e = 0; e < 4; e++) y[e] = fmaf(t[e], w, row[db][4 * q4 + e]) / merge.l;
      *(u32x2_t *)(orow + d0) = u32x2_t{pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])};
    }
}

// The tails of all rows: one (row, kv head) item per wavefront.
template <int HD, int G>
__global__ __launch_bounds__(256) void attn_tail_kernel(AttnArgs a) {
  constexpr int kQ = G * HD * 4, kWaveLds = kQ + kTailKeys * PartLds<bf16_t>::vrow(HD);
  __shared__ __attribute__((aligned(16))) unsigned char lds[4 * kWaveLds];
  const int w = threadIdx.x >> 6, item = (int)blockIdx.x * 4 + w;
  if (item >= a.rows * a.hkv) return;
  unsigned char *mine = lds + w * kWaveLds;
  attn_tail_body<bf16_t, HD, G>(a, item / a.hkv, item % a.hkv, threadIdx.x & 63, (float (*)[HD])mine, mine + kQ, true);
}

template <int HD, int G, int WAVES>
static hipError_t launch_chain(AttnArgs a, hipStream_t st) {
  constexpr int kLds = ChainLds<HD, WAVES>::total;
  static bool lds_allowed[64] = {};
  hipError_t e = allow_lds((const void *)attn_chain_kernel<HD, WAVES>, kLds, lds_allowed);
  if (e != hipSuccess) return e;
  const long long grid = (long long)a.hq * ((a.rows + WAVES * 32 - 1) / (WAVES * 32)), items = (long long)a.rows * a.hkv;
  if (grid > 0x7FFFFFFFll || items > 0x7FFFFFFFll) return hipErrorInvalidValue;
  a.max_parts = 1;                                            // the tail's partial is the only one
  hipLaunchKernelGGL((attn_tail_kernel<HD, G>), dim3((unsigned)((items + 3) / 4)), dim3(256), 0, st, a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((attn_chain_kernel<HD, WAVES>), dim3((unsigned)grid), dim3(WAVES * 64), kLds, st, a);
  return hipGetLastError();
}

// Which chains take attn_chain_kernel.  A workgroup of it walks all keys of its rows one block after the other, so its time grows
// with the keys alone until the chip is full; the hybrid path's grows with rows * heads * keys, and with few keys the
// fixed costs of its three launches and its partials count.  Crossing points measured in thousands of rows * heads, hybrid path faster below
// (32 heads of 128 on 32 and on 8 kv heads, 64 on 8, 40 on 40, 16 of 64): about 250 keys 5.5, 8, 8, 6, 4.5; 1050 keys 9, 10, 13, 10, 7.5; 2500 keys
// 13, 16, 17, 12, 10; 8700 keys 16, 18, 17.5, 16, 16.  us per call beside them, hybrid / chain: 192 rows of 32 heads alone 28.5 / 26.5, 320 rows 50 / 35, 512
// 78 / 48; at 768 keys before them 256 rows 52 / 60, 320 71 / 62; at 2048 384 rows 109 / 114, 512 148 / 121; at 8192 384 rows 261 / 330, 512 352 / 337,
// 768 533 / 352.  Tiles are 128 rows: below 192 rows (1.5 tiles) the hybrid path is never slower.
static bool chain_pays(int rows, int hq, int keys) {
  return rows >= 192 && (long long)rows * hq >= 4200 + 14400ll * keys / (keys + 1500);
}

template <typename T, int HD, int G>
static hipError_t launch_thg(AttnArgs a, int max_pos, hipStream_t st, AttnMerge *merge) {
  hipError_t e;
  if constexpr (sizeof(T) == 2) {
    if (attn_parts_covering(bulk_end(max_pos)) + 1 > a.max_parts) return hipErrorInvalidValue;
    if (a.anc == nullptr && chain_pays(a.rows, a.hq, max_pos + 1)) return launch_chain<HD, G, 4>(a, st);
    // hybrid: matrix-core bulk over [0, A(max_pos)) and the vector tail of every row in one launch
    a.tail_only = 1;
    a.bulk_keys = bulk_end(max_pos);
    a.bulk_blocks = (a.bulk_keys + 31) / 32;
    a.bulk_parts = attn_parts_covering(a.bulk_keys);
    const int rows = a.rows;
    for (int r0 = 0; r0 < rows; r0 += kPartialRows) {         // (more rows than the partials are planned for: a chain's)
      a.rows = std::min(kPartialRows, rows - r0);
      // At least four wavefronts per bulk workgroup, also for fewer than four blocks of 32 query rows: the ones
      // without rows still take their share of loading and staging the K/V blocks.
      const int qblocks = (a.rows * G + 31) / 32;
      if (qblocks <= 4) e = launch_hybrid<HD, G, 4>(a, 1, st);
      else e = launch_hybrid<HD, G, 8>(a, (qblocks + 7) / 8, st);
      if (e != hipSuccess) return e;
      if (merge != nullptr && rows <= kHeadRowsBf16 && a.bulk_parts + 1 <= kHeadMaxParts) {
        *merge = AttnMerge{a.part, a.max_parts, a.hq, HD, a.base, a.base_ptr, a.depth};
        return hipSuccess;
      }
      hipLaunchKernelGGL((attn_combine_kernel<T, HD>), dim3(a.rows, a.hq), dim3(HD), 0, st, a);
      e = hipGetLastError();
      if (e != hipSuccess) return e;
      a.q = (const float *)a.q + (size_t)a.rows * a.hq * HD;
      a.out = (T *)a.out + (size_t)a.rows * a.hq * HD;
      a.depth += a.rows;
      if (a.anc) a.anc += (size_t)a.rows * kAncStride;
    }
    return hipSuccess;
  } else {
    a.tail_only = 0;
    a.bulk_blocks = 0;
    const int n_parts = attn_parts_covering(max_pos + 1);
    if (n_parts > a.max_parts) return hipErrorInvalidValue;
    // (beyond one wavefront per SIMD the wavefronts of the two launches, with fewer registers and less LDS each, fill the chip better)
    if constexpr (HD * G <= 128) {                            // (more heads to a key head do not fit the registers)
      if (n_parts <= kRowParts && (long long)a.rows * a.hkv * n_parts <= 1024) {
        constexpr int kWaveLds = row_wave_bytes<HD, G>();
        static_assert(kRowParts * kWaveLds <= 158 * 1024, "a wavefront per part");
        static bool lds_allowed[64] = {};
        e = allow_lds((const void *)attn_row_kernel<HD, G>, kRowParts * kWaveLds, lds_allowed);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((attn_row_kernel<HD, G>), dim3(a.rows, a.hkv), dim3(n_parts * 64), n_parts * kWaveLds, st, a);
        return hipGetLastError();
      }
    }
    hipLaunchKernelGGL((attn_part_kernel<T, HD, G>), dim3(a.rows, a.hkv, n_parts), dim3(64), 0, st, a);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((attn_combine_kernel<T, HD>), dim3(a.rows, a.hq), dim3(HD), 0, st, a);
  return hipGetLastError();
}
template <typename T, int HD>
static hipError_t launch_th(const AttnArgs &a, int max_pos, hipStream_t st, AttnMerge *merge) {
  switch (a.hq / a.hkv) {
    case 1: return launch_thg<T, HD, 1>(a, max_pos, st, merge);
    case 2: return launch_thg<T, HD, 2>(a, max_pos, st, merge);
    case 4: return launch_thg<T, HD, 4>(a, max_pos, st, merge);
    case 8: return launch_thg<T, HD, 8>(a, max_pos, st, merge);
    default: return hipErrorInvalidValue;
  }
}

// max_pos: largest key position any row attends to (host-known bound: base + max depth).
hipError_t launch_attention(int dtype, const AttnArgs &args, int max_pos, hipStream_t st, AttnMerge *merge) {
  if (merge != nullptr) merge->part = nullptr;
  AttnArgs a = args;
  a.scale = (float)((double)a.scale * 1.4426950408889634);    // scores in units of log2
  if (a.rows < 1 || a.hkv < 1 || a.hq % a.hkv != 0) return hipErrorInvalidValue;
  if (a.raw.qkv != nullptr && (!attention_takes_raw(dtype, a.rows, a.hq, a.hkv) || a.raw.ldp % 4 || a.raw.split_stride % 4)) return hipErrorInvalidValue;
  if (a.hd == 128) return dtype == 1 ? launch_th<bf16_t, 128>(a, max_pos, st, merge) : launch_th<float, 128>(a, max_pos, st, merge);
  if (a.hd == 64) return dtype == 1 ? launch_th<bf16_t, 64>(a, max_pos, st, merge) : launch_th<float, 64>(a, max_pos, st, merge);
  return hipErrorInvalidValue;
}

hipError_t launch_attn_merge(const AttnMerge &m, int rows, void *out, hipStream_t st) {
  if (rows < 1 || (m.hd != 64 && m.hd != 128)) return hipErrorInvalidValue;
  AttnArgs a{};
  a.rows = rows; a.hq = m.hq; a.base = m.base; a.base_ptr = m.base_ptr; a.depth = m.depth;
  a.part = (float *)m.part; a.max_parts = m.max_parts; a.out = out; a.tail_only = 1;
  if (m.hd == 128) hipLaunchKernelGGL((attn_combine_kernel<bf16_t, 128>), dim3(rows, m.hq), dim3(128), 0, st, a);
  else hipLaunchKernelGGL((attn_combine_kernel<bf16_t, 64>), dim3(rows, m.hq), dim3(64), 0, st, a);
  return hipGetLastError();
}

}  // namespace spec
