// Training attention of harmonized context alignment (Sec. 3.2, appendix A.1) on the matrix cores.
//
// Streams m = 0 .. J-1 each hold keys/values for all T positions (stream 0 from the target's features,
// stream m from the draft features of training step m).  Query t (taken from stream J-1) sees
//   positions s <= t-(J-1)        from stream 0                      -> the "old" region, and
//   position  s  = t-o, o <= J-2  from stream J-1-o                  -> the "band": one key per stream.
// The old region is ordinary causal attention with the diagonal moved J-1 places and runs as a
// flash-attention loop over blocks of kBlockKeys keys staged in LDS.  The band is J-1 single keys per
// query, different for every query, and is folded in afterwards by the lanes that own the query.
//
// Work decomposition: a workgroup = 8 wavefronts = 256 (or 4 = 128) consecutive queries of one (batch, head); a wavefront
// owns 32 queries (one MFMA column block).  S^T = K Q^T and O^T = V^T P^T with v_mfma_f32_32x32x16_bf16, so a
// lane holds, for ITS query (lane % 32), 16 keys of every 32-key tile and 64 of the 128 output dims, and
// the softmax needs one exchange with lane ^ 32 only (by a permute of the vector unit; a query's two lanes add up their
// own sums and meet once, at the end).
// Bound: the serial chain of a block inside a wavefront (LDS reads, matrix instructions, maximum, exponentials), with two
// wavefronts per SIMD to cover each other; a wavefront's share of the staging is part of it and halves with 8 wavefronts.
// Measured (MI355X, us, launches back to back over one set of inputs): batch 2 x 2048, 32 heads of 128, three streams 115.7 -> 102 with 8
// wavefronts -> 98 with the band behind the loop (inputs from HBM: 113 both ways, 110 with its first rows asked for ahead of the last barrier); with 4: batch 2 x 1024 45.3 -> 43.3 (value rows read whole 1.5 of it, the maximum without a shuffle
// 0.3) -> 38.0.  Launches that leave the chip idle have a kernel of their own (hca_split_kernel).
// Tried: scores of the next block under the exponentials of this one, with keys and values copied straight into the LDS and transposed by the
// read (ds_read_b64_tr_b16): 84 -> 90 with one stream; without the exponentials that form would take 67, so the matrix cores' power limit is near.
#include "common.h"
#include "kernels.h"

namespace spec {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;

constexpr int kKeyTiles = 2;                  // 32-key MFMA tiles per staged block
constexpr int kBlockKeys = 32 * kKeyTiles;

__device__ __forceinline__ f32x16_t mfma16(const u32x4_t &a, const u32x4_t &b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}
__device__ __forceinline__ float lo_f32(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_f32(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

template <int HD, int WAVES> struct HcaLds {
  static constexpr int kstr = HD * 2 + 16;              // bytes per staged key row (+16: conflict-free b128 reads)
  static constexpr int vstr = kBlockKeys * 2 + 8;       // bytes per dim row of V^T (+8: conflict-free b64 reads)
  // A wavefront stages whole value rows (HD / 8 lanes a row, 512 / HD key pairs), eight dims a lane: the lanes of dims 32
  // apart would store to the same banks, so every 32 dims start 512 / HD words further on.
  static constexpr int vpad = 512 / HD * 4;
  static constexpr int buf = kBlockKeys * kstr + HD * vstr + HD / 32 * vpad;
  static constexpr int brow = HD * 2 + 16;              // band scratch: bytes per key (or value) row
  static constexpr int bwave = 2 * 32 * brow;           // ... per wavefront: 32 key rows + 32 value rows
  static constexpr int total = 2 * buf > WAVES * bwave ? 2 * buf : WAVES * bwave;   // main loop double-buffered
};

// Orders this wavefront's LDS writes before its later LDS reads of other lanes' data.  The LDS executes
// one wavefront's operations in issue order, so only the compiler has to be kept from reordering them.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Workgroup id -> (batch, kv head, head of the group, query tile).  Ids 8 apart run on one XCD: all tiles and heads that
// read the same keys/values are placed there.  An XCD's (batch, kv head) groups are taken in chunks of up to kHcaChunk;
// inside a chunk the workgroups go LONGEST TILE FIRST across its groups (the causal mask makes the last tile the
// longest, and a launch of a few workgroups per slot ends when its last long tile does), the heads of one group next to
// each other so that they share the keys and values through L2.  The chunk bounds the keys and values in use at a time:
// tile-major order over 64 groups per XCD (batch 16) runs at 490 TFLOP/s where group-major order reaches 659; over the
// 8 groups of the batch-2 launch it is 23 % faster than group-major.  (With a number of groups that is not a multiple
// of 8 the XCD placement would leave XCDs idle or uneven; the ids then run chunk by chunk over all groups.)
constexpr int kHcaChunk = 8;
struct Place { int qt, gh, bi, hk; };
__device__ __forceinline__ Place place(const HcaArgs &a, int rows, int chunk_most = kHcaChunk) {   // rows: queries per workgroup
  const int G = a.hq / a.hkv;
  const int n_qt = (a.seq + rows - 1) / rows;
  const int n_grp = a.batch * a.hkv;
  const bool affine = (n_grp & 7) == 0;
  const int grp_per_list = affine ? n_grp >> 3 : n_grp;      // groups whose workgroups form one ordered list
  const int r_id = affine ? (int)blockIdx.x >> 3 : (int)blockIdx.x;
  const int chunk_wgs = chunk_most * G * n_qt;               // workgroups of a full chunk
  const int chunk = r_id / chunk_wgs, in_chunk = r_id % chunk_wgs;
  const int chunk_grps = min(chunk_most, grp_per_list - chunk * chunk_most);   // the last chunk may be short
  const int qt = n_qt - 1 - in_chunk / (chunk_grps * G);
  const int in_tile = in_chunk % (chunk_grps * G);
  const int gh = in_tile % G;
  const int grp_local = chunk * chunk_most + in_tile / G;
  const int grp = affine ? grp_local * 8 + ((int)blockIdx.x & 7) : grp_local;
  return Place{qt, gh, grp / a.hkv, grp % a.hkv};
}

template <int HD, int WAVES>
__global__ __launch_bounds__(WAVES * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void hca_attention_kernel(HcaArgs a) {
  using L = HcaLds<HD, WAVES>;
  constexpr int NT = WAVES * 64, ROWS = WAVES * 32;   // threads, queries per workgroup
  constexpr int DB = HD / 32;                 // 32-dim blocks of the output
  constexpr int KK = HD / 16;                 // MFMA steps of q.k
  constexpr int PPR = HD * 2 / 16;            // 16-byte pieces per key row
  constexpr int KP = kBlockKeys * PPR / NT;          // K pieces per thread per block
  // The band's first rows are asked for ahead of the barrier behind the last key block, which a wavefront that sees nothing of that block reaches
  // early (see the band below)
  constexpr bool kAskEarly = WAVES == 8;
  constexpr int VP = kBlockKeys / 2 * PPR / NT;      // V (key pair, piece) items per thread per block
  static_assert(kBlockKeys * PPR % NT == 0 && (kBlockKeys / 2 * PPR) % NT == 0, "staging split");
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];

  const Place at = place(a, ROWS);
  const int qt = at.qt, gh = at.gh, bi = at.bi, hk = at.hk, G = a.hq / a.hkv;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), c = lane & 31, g = lane >> 5;
  const int T = a.seq, J = a.n_streams;
  const float c2 = a.scale_log2e;
  const size_t kv_stride = (size_t)a.hkv * HD;                // elements between consecutive positions
  const size_t kv_off = (size_t)bi * T * kv_stride + (size_t)hk * HD;
  const bf16_t *kg = (const bf16_t *)a.k[0] + kv_off;
  const bf16_t *vg = (const bf16_t *)a.v[0] + kv_off;

  const int r0 = qt * ROWS + wave * 32;   // first query of the wavefront
  const int t = r0 + c;
  const int tq = min(t, T - 1);               // queries past the end compute on the last one and are not stored
  const int lim = tq - (J - 1);               // last old-region key of this query (may be negative: none)
  const int wg_lim = min(qt * ROWS + ROWS - 1, T - 1) - (J - 1);
  const int nb = wg_lim >= 0 ? wg_lim / kBlockKeys + 1 : 0;
  const int wave_lim = min(r0 + 31, T - 1) - (J - 1);

  // Per-thread byte offsets of its pieces inside a key block, computed once; a block's loads are then a
  // uniform base plus these.  Only a block that reaches past the sequence end needs per-key clamping
  // (keys past the end are masked for every query; they are read from the last position).
  constexpr uint32_t kEsz = 2;
  uint32_t koff[KP], voff[VP];
#pragma unroll
  for (int e = 0; e < KP; e++) {
    const int q = tid + e * NT;
    koff[e] = (uint32_t)((q / PPR) * kv_stride + (q % PPR) * 8) * kEsz;
  }
#pragma unroll
  for (int e = 0; e < VP; e++) {
    const int q = tid + e * NT;
    voff[e] = (uint32_t)((2 * (q / PPR)) * kv_stride + (q % PPR) * 8) * kEsz;
  }
  const uint32_t row_bytes = (uint32_t)kv_stride * kEsz;
  u32x4_t kreg[KP], vreg[VP][2];
  auto prefetch = [&](int blk) {
    const size_t blk_off = (size_t)blk * kBlockKeys * row_bytes;
    const unsigned char *kbase = (const unsigned char *)kg + blk_off, *vbase = (const unsigned char *)vg + blk_off;
    if (blk * kBlockKeys + kBlockKeys <= T) {
#pragma unroll
      for (int e = 0; e < KP; e++) kreg[e] = *(const u32x4_t *)(kbase + koff[e]);
#pragma unroll
      for (int e = 0; e < VP; e++) {
        vreg[e][0] = *(const u32x4_t *)(vbase + voff[e]);
        vreg[e][1] = *(const u32x4_t *)(vbase + voff[e] + row_bytes);
      }
    } else {
#pragma unroll
      for (int e = 0; e < KP; e++) {
        const int q = tid + e * NT;
        const int key = min(blk * kBlockKeys + q / PPR, T - 1);
        kreg[e] = *(const u32x4_t *)(kg + (size_t)key * kv_stride + (q % PPR) * 8);
      }
#pragma unroll
      for (int e = 0; e < VP; e++) {
        const int q = tid + e * NT;
        const int pair = q / PPR, piece = q % PPR;
        const int key0 = min(blk * kBlockKeys + 2 * pair, T - 1), key1 = min(blk * kBlockKeys + 2 * pair + 1, T - 1);
        vreg[e][0] = *(const u32x4_t *)(vg + (size_t)key0 * kv_stride + piece * 8);
        vreg[e][1] = *(const u32x4_t *)(vg + (size_t)key1 * kv_stride + piece * 8);
      }
    }
  };
  auto stage = [&](int buf) {
    unsigned char *k_lds = lds + buf * L::buf, *vt_lds = k_lds + kBlockKeys * L::kstr;
#pragma unroll
    for (int e = 0; e < KP; e++) {
      const int q = tid + e * NT;
      *(u32x4_t *)(k_lds + (q / PPR) * L::kstr + (q % PPR) * 16) = kreg[e];
    }
#pragma unroll
    for (int e = 0; e < VP; e++) {                            // V^T[dim][key], two keys per 32-bit store
      const int q = tid + e * NT;
      const int pair = q / PPR, piece = q % PPR;
      const uint32_t w0[4] = {vreg[e][0].x, vreg[e][0].y, vreg[e][0].z, vreg[e][0].w};
      const uint32_t w1[4] = {vreg[e][1].x, vreg[e][1].y, vreg[e][1].z, vreg[e][1].w};
#pragma unroll
      for (int d2 = 0; d2 < 8; d2++) {
        const uint32_t x = (d2 & 1) ? ((w0[d2 >> 1] >> 16) | (w1[d2 >> 1] & 0xFFFF0000u))
                                    : ((w0[d2 >> 1] & 0xFFFFu) | (w1[d2 >> 1] << 16));
        *(uint32_t *)(vt_lds + (piece * 8 + d2) * L::vstr + (piece >> 2) * L::vpad + pair * 4) = x;
      }
    }
  };

  // V^T fragment (A operand) of 16-key step st = 2*tile + half and dim block db: keys step*16 + 4g + {0..3, 8..11}
  auto vread = [&](const unsigned char *vt_lds, int st, int db) {
    const unsigned char *vp = vt_lds + (db * 32 + c) * L::vstr + db * L::vpad + (16 * st + 4 * g) * 2;
    const u32x2_t v0 = *(const u32x2_t *)vp, v1 = *(const u32x2_t *)(vp + 16);
    return u32x4_t{v0.x, v0.y, v1.x, v1.y};
  };

  // query fragments (B operand): step kk covers dims kk*16 + g*8 .. +8 of query c.  They are requested before
  // the first key block: loads complete in order, so once that block has arrived nothing in
  // the main loop waits on the memory counter for the queries' sake (such a wait would also stall on the
  // block in flight).
  const bf16_t *qrow = (const bf16_t *)a.q + (((size_t)bi * T + tq) * a.hq + (size_t)hk * G + gh) * HD;
  u32x4_t qf[KK];
#pragma unroll
  for (int kk = 0; kk < KK; kk++) qf[kk] = *(const u32x4_t *)(qrow + kk * 16 + g * 8);

  f32x16_t o[DB];
#pragma unroll
  for (int db = 0; db < DB; db++)
#pragma unroll
    for (int v = 0; v < 16; v++) o[db][v] = 0.f;
  // running maximum (of score * scale * log2 e) and sum of 2^(score' - maximum)
  float m_run = -INFINITY, l_run = 0.f;

  if (nb > 0) {
    prefetch(0);
    stage(0);
    __syncthreads();
    if (nb > 1) prefetch(1);
  }
  for (int blk = 0; blk < nb; blk++) {
    const int cur = blk & 1;
    const unsigned char *k_lds = lds + cur * L::buf, *vt_lds = k_lds + kBlockKeys * L::kstr;
    const bool act = blk * kBlockKeys <= wave_lim;            // wavefront-uniform: some query here sees this block
    // The next block is staged first (into the buffer every wavefront left at the last barrier), from the
    // registers its loads filled during the previous iteration; the loads of the block after it follow.
    if (blk + 1 < nb) {
      stage(cur ^ 1);
      if (blk + 2 < nb) prefetch(blk + 2);
    }
    if (act) {
      f32x16_t s[kKeyTiles];
#pragma unroll
      for (int kt = 0; kt < kKeyTiles; kt++) {
#pragma unroll
        for (int v = 0; v < 16; v++) s[kt][v] = 0.f;
#pragma unroll
        for (int kk = 0; kk < KK; kk++) {
          const u32x4_t kf = *(const u32x4_t *)(k_lds + (kt * 32 + c) * L::kstr + kk * 32 + g * 16);
          s[kt] = mfma16(kf, qf[kk], s[kt]);
        }
      }
      // s[kt][v] = q . k for key blk*kBlockKeys + kt*32 + 8*(v/4) + 4*g + v%4 and query c
      if (blk * kBlockKeys + kBlockKeys - 1 > r0 - (J - 1)) {  // the block reaches past some query's region
        const int key0 = blk * kBlockKeys + 4 * g;
#pragma unroll
        for (int kt = 0; kt < kKeyTiles; kt++)
#pragma unroll
          for (int v = 0; v < 16; v++)
            if (key0 + kt * 32 + 8 * (v >> 2) + (v & 3) > lim) s[kt][v] = -INFINITY;
      }
      float mb = -INFINITY;
#pragma unroll
      for (int kt = 0; kt < kKeyTiles; kt++)
#pragma unroll
        for (int v = 0; v < 16; v++) mb = fmaxf(mb, s[kt][v]);
      mb = max_halves(mb);
      // The reference maximum moves only when the block's maximum exceeds it by more than 2^8: until then
      // the probabilities are taken against the old reference (at most 2^8, harmless in fp32 and bf16, and
      // the final division by the sum cancels the choice), and the 64 output registers are left alone.
      const float mb2 = mb * c2;
      const bool move = mb2 > m_run + 8.f;                     // also the first finite maximum after -inf
      if (__any(move)) {
        const float m_new = move ? mb2 : m_run;
        const float corr = move ? __builtin_amdgcn_exp2f(m_run - m_new) : 1.f;   // m_new is finite where move
        l_run *= corr;
        m_run = m_new;
#pragma unroll
        for (int db = 0; db < DB; db++)
#pragma unroll
          for (int v = 0; v < 16; v++) o[db][v] *= corr;
      }
      const float m_use = m_run == -INFINITY ? 0.f : m_run;    // nothing seen yet: every term below becomes 0
      // Per 32-key tile: probabilities (vector ALU), then O^T += V^T P^T in two 16-key steps (matrix cores);
      // step (kt, h) uses the lane's own values v = 8h .. 8h+7 of tile kt, i.e. keys kt*32 + 16h + 8*(e/4) + 4g
      // + e%4, and V^T supplies the same keys per dim.  The tiles are independent, so the second tile's
      // vector arithmetic can run while the first tile's matrix instructions execute.
      float ls = 0.f;
#pragma unroll
      for (int kt = 0; kt < kKeyTiles; kt++) {
        float p[16];
        uint32_t pk[8];                                       // probabilities, two bf16 per word
#pragma unroll
        for (int v = 0; v < 16; v++) { p[v] = __builtin_amdgcn_exp2f(fmaf(s[kt][v], c2, -m_use)); ls += p[v]; }
#pragma unroll
        for (int e = 0; e < 8; e++) pk[e] = pack_bf16x2(p[2 * e], p[2 * e + 1]);
#pragma unroll
        for (int h = 0; h < 2; h++) {
          const u32x4_t pf = {pk[4 * h], pk[4 * h + 1], pk[4 * h + 2], pk[4 * h + 3]};
#pragma unroll
          for (int db = 0; db < DB; db++) o[db] = mfma16(vread(vt_lds, 2 * kt + h, db), pf, o[db]);
        }
      }
      l_run += ls;
    }
    if (kAskEarly && blk + 1 == nb) break;
    __syncthreads();                                          // block blk+1 staged; everyone is done with block blk
  }

  // The band last: key t-off of stream J-1-off, off = J-2 .. 0.  These rows are read once, from HBM (67 MB a stream at batch 2 x 2048, 32
  // heads); ahead of the loop all workgroups of the launch asked for them at the same time and the matrix cores waited, behind it they ask as
  // they finish, under the others' blocks (three of 1000 positions, 8 heads, eight streams 41.7 -> 38.4 us, one of 852, 32 heads, five 34.0 ->
  // 31.6; a single short workgroup per compute unit gains nothing, 608 positions of 4 heads 21.9 -> 22.1).  Many workgroups of heads that share their
  // rows through the L2 lose by it: head dim 64, 64 heads on 8, two of 1024 positions 36.1 -> 37.4.  A workgroup of 8 wavefronts has the compute unit
  // to itself and waits alone for its first rows; they are asked for ahead of the last barrier: 64 heads on 16, one of 2048 positions 98.6 -> 94.3 (96.5
  // with the band ahead of the loop), 32 heads on 8, two of 2000, five streams 110.1 -> 108.2 (104.7).  With 4 wavefronts that pays
  // for some (one of 2048 positions, 32 heads 64.1 -> 62.3) and costs others more (two of 1024 41.1 -> 43.4).
  // The 32 queries of the wavefront need 32 consecutive rows of a stream: they are read with coalesced
  // 16-byte accesses (a row = PPR lanes) into the wavefront's own LDS area, and then every lane pair (c, c+32) picks up the row of ITS query,
  // splitting the dot product by the dims of its query fragments and the value row by the dims of its output registers.  No other wavefront is
  // involved (every one has left the key blocks' LDS at the last barrier); the next stream's rows travel while one's are used.
  {
    unsigned char *bk = lds + wave * L::bwave, *bv = bk + 32 * L::brow;
    constexpr int BP = 32 * PPR / 64;                         // 16-byte pieces per lane per tensor
    u32x4_t kw_[BP], vw_[BP];
    auto fetch = [&](int off) __attribute__((always_inline)) {
      const bf16_t *kb = (const bf16_t *)a.k[J - 1 - off] + kv_off;
      const bf16_t *vb = (const bf16_t *)a.v[J - 1 - off] + kv_off;
#pragma unroll
      for (int e = 0; e < BP; e++) {
        const int idx = lane + 64 * e;
        const int row = min(max(r0 + idx / PPR - off, 0), T - 1);
        kw_[e] = *(const u32x4_t *)(kb + (size_t)row * kv_stride + (idx % PPR) * 8);
        vw_[e] = *(const u32x4_t *)(vb + (size_t)row * kv_stride + (idx % PPR) * 8);
      }
    };
    if (J > 1) {
      fetch(J - 2);
      if (kAskEarly) __syncthreads();                         // everyone is done with the key blocks
    }
    for (int off = J - 2; off >= 0; off--) {
#pragma unroll
      for (int e = 0; e < BP; e++) {
        const int idx = lane + 64 * e;
        *(u32x4_t *)(bk + (idx / PPR) * L::brow + (idx % PPR) * 16) = kw_[e];
        *(u32x4_t *)(bv + (idx / PPR) * L::brow + (idx % PPR) * 16) = vw_[e];
      }
      if (off > 0) fetch(off - 1);                            // on their way while this stream's rows are used
      wave_lds_order();
      const bool have = tq - off >= 0;
      float dot = 0.f;
#pragma unroll
      for (int kk = 0; kk < KK; kk++) {
        const u32x4_t kw = *(const u32x4_t *)(bk + c * L::brow + kk * 32 + g * 16);
        const uint32_t kx[4] = {kw.x, kw.y, kw.z, kw.w}, qx[4] = {qf[kk].x, qf[kk].y, qf[kk].z, qf[kk].w};
#pragma unroll
        for (int e = 0; e < 4; e++) {
          dot = fmaf(lo_f32(qx[e]), lo_f32(kx[e]), dot);
          dot = fmaf(hi_f32(qx[e]), hi_f32(kx[e]), dot);
        }
      }
      dot += __shfl_xor(dot, 32, 64);
      const float sc = have ? dot * c2 : -INFINITY;
      const float m_new = fmaxf(m_run, sc);
      const float m_use = m_new == -INFINITY ? 0.f : m_new;
      const float corr = __builtin_amdgcn_exp2f(m_run - m_use);
      const float p = have ? __builtin_amdgcn_exp2f(sc - m_use) : 0.f;
      l_run = fmaf(l_run, corr, g == 0 ? p : 0.f);             // the two lanes of a query add up their sums at the end
      m_run = m_new;
#pragma unroll
      for (int db = 0; db < DB; db++)
#pragma unroll
        for (int q4 = 0; q4 < 4; q4++) {
          const u32x2_t vw = *(const u32x2_t *)(bv + c * L::brow + (db * 32 + 8 * q4 + 4 * g) * 2);
          o[db][4 * q4 + 0] = fmaf(p, lo_f32(vw.x), o[db][4 * q4 + 0] * corr);
          o[db][4 * q4 + 1] = fmaf(p, hi_f32(vw.x), o[db][4 * q4 + 1] * corr);
          o[db][4 * q4 + 2] = fmaf(p, lo_f32(vw.y), o[db][4 * q4 + 2] * corr);
          o[db][4 * q4 + 3] = fmaf(p, hi_f32(vw.y), o[db][4 * q4 + 3] * corr);
        }
      wave_lds_order();                                       // the next stream's rows overwrite the area
    }
  }

  const float inv = 1.f / (l_run + __shfl_xor(l_run, 32, 64));
  if (t >= T) return;
  bf16_t *orow = (bf16_t *)a.out + (((size_t)bi * T + t) * a.hq + (size_t)hk * G + gh) * HD;
#pragma unroll
  for (int db = 0; db < DB; db++)
#pragma unroll
    for (int q4 = 0; q4 < 4; q4++) {
      u32x2_t w;
      w.x = pack_bf16x2(o[db][4 * q4 + 0] * inv, o[db][4 * q4 + 1] * inv);
      w.y = pack_bf16x2(o[db][4 * q4 + 2] * inv, o[db][4 * q4 + 3] * inv);
      *(u32x2_t *)(orow + db * 32 + 8 * q4 + 4 * g) = w;
    }
}

// ---- launches that leave the chip idle ------------------------------------------------------------
// A workgroup = 4 wavefronts and 32 queries; the wavefronts share out the KEYS, a block of kBlockKeys each a round, and do what hca_attention_kernel
// does, operation by operation: a sequence's outputs have the same bits in a launch of any size.  What does not depend on the blocks before is
// done side by side: a block's scores and their maximum.  The chain of references runs through the maxima of a round's blocks, every wavefront
// for itself, and with its own block's reference a wavefront forms the probabilities and their sum.  What is left in the blocks' order is
// O^T += V^T P^T, and there the output's 32-dim parts do not depend on each other: wavefront db takes a round's blocks one after the other for dims
// 32 db .. from the LDS (probabilities as fragments, value rows as they are, transposed by the read).  The band's products with the queries are
// formed ahead, a stream a wavefront, and its value rows wait in the LDS.  A 128-query tile's chain of T / 64 blocks becomes one of T / 256 rounds on
// four times as many workgroups; the price is that every 32 queries load their keys and values themselves, so it is only for launches that do not
// fill the chip (split_pays).
// Bound: latency up to 300 positions (launch, first rows, two barriers a round), then the way of a round's 256 keys from the L2 with nothing of the next
// round under it: requested ahead they spill at head dim 128 (2048 positions 33 -> 42 us) and gain nothing at 64.  Four heads of 128, 2048 positions, three
// streams 51.7 -> 33.2 us (hca_attention_kernel / this); 333 positions, 16 heads of 64, two streams 9.8 -> 7.1.  Wavefronts with a softmax of their own that merge at the end need no
// rounds, 25.5 and 6.0, but add up in another order: a sequence then differed by rounding (1.6e-3) with the number of sequences and heads beside it.
// Eight wavefronts in halves: 31.9 and 6.9, 256 positions of 32 heads 7.3 -> 8.2.
// (each rounded by itself: hca_attention_kernel multiplies in a branch of its own)
__device__ __forceinline__ float turn_add(float l, float turn, float ls) {
#pragma clang fp contract(off)
  const float x = l * turn;
  return x + ls;
}

constexpr int kSplitWaves = 4;
template <int HD> struct SplitLds {
  static constexpr int vals = kBlockKeys * HD * 2;      // a block's value rows
  static constexpr int probs = 32 * kBlockKeys * 2;     // ... and probabilities
  static constexpr int probs0 = kSplitWaves * vals;     // (of a round's blocks)
  static constexpr int max0 = probs0 + kSplitWaves * probs;   // two sets (rounds alternate) of the blocks' maxima, [block][query] ..
  static constexpr int sum0 = max0 + 2 * kSplitWaves * 32 * 4;    // .. and sums, [block][lane]
  static constexpr int score0 = sum0 + 2 * kSplitWaves * 64 * 4;  // the band's scores, [stream][query]
  static constexpr int band0 = score0 + (kMaxStreams - 1) * 32 * 4;   // ... and value rows, [stream][query]
  static constexpr int brow = HD * 2 + 16;
  static constexpr int total(int streams) { return band0 + (streams - 1) * 32 * brow; }
};

template <int HD>
__global__ __launch_bounds__(kSplitWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void hca_split_kernel(HcaArgs a) {
  using L = SplitLds<HD>;
  constexpr int W = kSplitWaves, DB = HD / 32, KK = HD / 16, PPR = HD * 2 / 16, VP = kBlockKeys * PPR / 64, BP = 32 * PPR / 64;
  static_assert(DB <= W, "a wavefront per 32 dims");
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const Place at = place(a, 32, a.batch * a.hkv);             // (few workgroups: one list, longest tile first)
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), c = lane & 31, g = lane >> 5;
  const int T = a.seq, J = a.n_streams, G = a.hq / a.hkv;
  const float c2 = a.scale_log2e;
  const size_t kv_stride = (size_t)a.hkv * HD, kv_off = (size_t)at.bi * T * kv_stride + (size_t)at.hk * HD;
  const bf16_t *kg = (const bf16_t *)a.k[0] + kv_off, *vg = (const bf16_t *)a.v[0] + kv_off;
  const int r0 = at.qt * 32, t = r0 + c, tq = min(t, T - 1);  // queries past the end compute on the last one and are not stored
  const int lim = tq - (J - 1);
  const int last = min(r0 + 31, T - 1) - (J - 1);             // last old-region key of any query
  const int nb = last >= 0 ? last / kBlockKeys + 1 : 0;
  const size_t q_off = (((size_t)at.bi * T + tq) * a.hq + (size_t)at.hk * G + at.gh) * HD;
  float *const max_sh = (float *)(lds + L::max0), *const sum_sh = (float *)(lds + L::sum0), *const score_sh = (float *)(lds + L::score0);
  u32x4_t qf[KK], kf[kKeyTiles][KK], vr[VP];
#pragma unroll
  for (int kk = 0; kk < KK; kk++) qf[kk] = *(const u32x4_t *)((const bf16_t *)a.q + q_off + kk * 16 + g * 8);

  // A block's loads are a uniform base and 32-bit offsets (a launch of few workgroups has few heads).  Keys past the end are the last one, masked.
  const uint32_t row_bytes = (uint32_t)kv_stride * 2;
  auto load_k = [&](int blk) __attribute__((always_inline)) {
    const unsigned char *const base = (const unsigned char *)(kg + (size_t)blk * kBlockKeys * kv_stride);
    const int most = T - 1 - blk * kBlockKeys;
#pragma unroll
    for (int kt = 0; kt < kKeyTiles; kt++) {
      const uint32_t row = (uint32_t)min(kt * 32 + c, most) * row_bytes + g * 16;
#pragma unroll
      for (int kk = 0; kk < KK; kk++) kf[kt][kk] = *(const u32x4_t *)(base + row + kk * 32);
    }
  };
  auto load_v = [&](int blk) __attribute__((always_inline)) {
    const unsigned char *const base = (const unsigned char *)(vg + (size_t)blk * kBlockKeys * kv_stride);
    const int most = T - 1 - blk * kBlockKeys;
#pragma unroll
    for (int e = 0; e < VP; e++) vr[e] = *(const u32x4_t *)(base + ((uint32_t)min(lane / PPR + e * (64 / PPR), most) * row_bytes + lane % PPR * 16));
  };

  // the band: key tq - off of stream J-1-off for every query, off = J-2 .. 0.  A lane pair shares the product by the dims of its query fragments.
  for (int off = W - 1 - wave; off <= J - 2; off += W) {      // (the last wavefronts first: they have the fewest blocks)
    const bf16_t *kb = (const bf16_t *)a.k[J - 1 - off] + kv_off, *vb = (const bf16_t *)a.v[J - 1 - off] + kv_off;
    u32x4_t bk[KK], bv[BP];
#pragma unroll
    for (int kk = 0; kk < KK; kk++) bk[kk] = *(const u32x4_t *)(kb + (size_t)max(tq - off, 0) * kv_stride + kk * 16 + g * 8);
#pragma unroll
    for (int e = 0; e < BP; e++) {
      const int idx = lane + 64 * e;
      bv[e] = *(const u32x4_t *)(vb + (size_t)min(max(r0 + idx / PPR - off, 0), T - 1) * kv_stride + (idx % PPR) * 8);
    }
    float dot = 0.f;
#pragma unroll
    for (int kk = 0; kk < KK; kk++) {
      const uint32_t kx[4] = {bk[kk].x, bk[kk].y, bk[kk].z, bk[kk].w}, qx[4] = {qf[kk].x, qf[kk].y, qf[kk].z, qf[kk].w};
#pragma unroll
      for (int e = 0; e < 4; e++) {
        dot = fmaf(lo_f32(qx[e]), lo_f32(kx[e]), dot);
        dot = fmaf(hi_f32(qx[e]), hi_f32(kx[e]), dot);
      }
    }
    dot += __shfl_xor(dot, 32, 64);
    if (g == 0) score_sh[off * 32 + c] = tq - off >= 0 ? dot * c2 : -INFINITY;
#pragma unroll
    for (int e = 0; e < BP; e++) {
      const int idx = lane + 64 * e;
      *(u32x4_t *)(lds + L::band0 + (off * 32 + idx / PPR) * L::brow + (idx % PPR) * 16) = bv[e];
    }
  }

  f32x16_t o;                                                 // dims 32 wave .. of this wavefront's part of the output
#pragma unroll
  for (int v = 0; v < 16; v++) o[v] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  const int vlane = value_lane<HD>(lane);
  for (int b0 = 0, set = 0; b0 < nb; b0 += W, set ^= 1) {
    const int blk = b0 + wave;
    const bool live = blk < nb;
    f32x16_t s[kKeyTiles];
    float mb2 = -INFINITY;
    if (live) {
      load_k(blk);
      load_v(blk);
#pragma unroll
      for (int kt = 0; kt < kKeyTiles; kt++) {
#pragma unroll
        for (int v = 0; v < 16; v++) s[kt][v] = 0.f;
#pragma unroll
        for (int kk = 0; kk < KK; kk++) s[kt] = mfma16(kf[kt][kk], qf[kk], s[kt]);
      }
      // s[kt][v] = q . k for key blk*kBlockKeys + kt*32 + 8*(v/4) + 4*g + v%4 and query c
      if (blk * kBlockKeys + kBlockKeys - 1 > r0 - (J - 1)) {  // the block reaches past some query's region
        const int key0 = blk * kBlockKeys + 4 * g;
#pragma unroll
        for (int kt = 0; kt < kKeyTiles; kt++)
#pragma unroll
          for (int v = 0; v < 16; v++)
            if (key0 + kt * 32 + 8 * (v >> 2) + (v & 3) > lim) s[kt][v] = -INFINITY;
      }
      float mb = -INFINITY;
#pragma unroll
      for (int kt = 0; kt < kKeyTiles; kt++)
#pragma unroll
        for (int v = 0; v < 16; v++) mb = fmaxf(mb, s[kt][v]);
      mb2 = max_halves(mb) * c2;
    }
    if (g == 0) max_sh[(set * W + wave) * 32 + c] = mb2;
    __syncthreads();                                          // the round's maxima are there, and the round before is used up

    // the chain of references: a block's moves it by more than 2^8 only (as in hca_attention_kernel)
    float corr[W], m_own = -INFINITY;
#pragma unroll
    for (int j = 0; j < W; j++) {
      const float mbj = max_sh[(set * W + j) * 32 + c];
      const bool move = mbj > m_run + 8.f;
      const float m_new = move ? mbj : m_run;
      corr[j] = move ? __builtin_amdgcn_exp2f(m_run - m_new) : 1.f;
      m_run = m_new;
      if (j == wave) m_own = m_run;
    }
    uint32_t pk[kKeyTiles * 8];                               // probabilities, two bf16 per word
    if (live) {
      const float m_use = m_own == -INFINITY ? 0.f : m_own;   // nothing seen yet: every term below becomes 0
      float ls = 0.f;
#pragma unroll
      for (int kt = 0; kt < kKeyTiles; kt++) {
        float p[16];
#pragma unroll
        for (int v = 0; v < 16; v++) { p[v] = __builtin_amdgcn_exp2f(fmaf(s[kt][v], c2, -m_use)); ls += p[v]; }
#pragma unroll
        for (int e = 0; e < 8; e++) pk[kt * 8 + e] = pack_bf16x2(p[2 * e], p[2 * e + 1]);
      }
      sum_sh[(set * W + wave) * 64 + lane] = ls;
      unsigned char *const vals = lds + wave * L::vals, *const probs = lds + L::probs0 + wave * L::probs + lane * 16;
#pragma unroll
      for (int e = 0; e < VP; e++) {
        const int idx = lane + 64 * e, row = idx / PPR, piece = idx % PPR;
        *(u32x4_t *)(vals + value_piece<HD>(row, piece)) = vr[e];
      }
#pragma unroll
      for (int st = 0; st < 4; st++) *(u32x4_t *)(probs + st * 1024) = u32x4_t{pk[4 * st], pk[4 * st + 1], pk[4 * st + 2], pk[4 * st + 3]};
    }
    __syncthreads();
    if (wave >= DB) continue;
#pragma unroll
    for (int j = 0; j < W; j++) {
      if (b0 + j >= nb) break;
      l_run = turn_add(l_run, corr[j], sum_sh[(set * W + j) * 64 + lane]);
      const unsigned char *const vals = lds + j * L::vals, *const probs = lds + L::probs0 + j * L::probs + lane * 16;
#pragma unroll
      for (int v = 0; v < 16; v++) o[v] *= corr[j];
#pragma unroll
      for (int st = 0; st < 4; st++)                          // 16 keys
        o = mfma16(value_fragment<HD>(vals, vlane, wave, 16 * st), *(const u32x4_t *)(probs + st * 1024), o);
    }
  }
  if (nb == 0) __syncthreads();                               // the band is there
  if (wave >= DB) return;
  for (int off = J - 2; off >= 0; off--) {
    const float sc = score_sh[off * 32 + c];
    const float m_new = fmaxf(m_run, sc);
    const float m_use = m_new == -INFINITY ? 0.f : m_new;
    const float corr = __builtin_amdgcn_exp2f(m_run - m_use);
    const float p = tq - off >= 0 ? __builtin_amdgcn_exp2f(sc - m_use) : 0.f;
    l_run = fmaf(l_run, corr, g == 0 ? p : 0.f);              // the two lanes of a query add up their sums at the end
    m_run = m_new;
#pragma unroll
    for (int q4 = 0; q4 < 4; q4++) {
      const u32x2_t vw = *(const u32x2_t *)(lds + L::band0 + (off * 32 + c) * L::brow + (wave * 32 + 8 * q4 + 4 * g) * 2);
      o[4 * q4 + 0] = fmaf(p, lo_f32(vw.x), o[4 * q4 + 0] * corr);
      o[4 * q4 + 1] = fmaf(p, hi_f32(vw.x), o[4 * q4 + 1] * corr);
      o[4 * q4 + 2] = fmaf(p, lo_f32(vw.y), o[4 * q4 + 2] * corr);
      o[4 * q4 + 3] = fmaf(p, hi_f32(vw.y), o[4 * q4 + 3] * corr);
    }
  }
  const float inv = 1.f / (l_run + __shfl_xor(l_run, 32, 64));
  if (t >= T) return;
  bf16_t *const orow = (bf16_t *)a.out + q_off + wave * 32;
#pragma unroll
  for (int q4 = 0; q4 < 4; q4++) {
    u32x2_t w;
    w.x = pack_bf16x2(o[4 * q4 + 0] * inv, o[4 * q4 + 1] * inv);
    w.y = pack_bf16x2(o[4 * q4 + 2] * inv, o[4 * q4 + 3] * inv);
    *(u32x2_t *)(orow + 8 * q4 + 4 * g) = w;
  }
}

// Workgroups of 8 wavefronts save staging, but a tile of 256 has more rows past the end of the sequence, and a compute unit holds one
// where it holds two of 4 wavefronts, so that the order longest first evens out less.  They pay
//  * without a half-empty tile (an even number of 128-query tiles): 512 workgroups of 2000 positions 110 -> 104 us, of 1920 102 -> 101; 448 of
//    2000 102 -> 97, of 1920 94 -> 96; 1024 of 2000 220 -> 204, of 1920 199 -> 202;
//  * from 1700 positions on (14 tiles): 448 of 1700 92 -> 85, of 1792 94 -> 87; 480 of 1536 109 -> 108 and 92 -> 100, 400 of 1280 87 -> 88 and
//    70 -> 78, but also 384 of 1536 77 -> 70 and 68 -> 61;
//  * with 400 to 512 workgroups, a long and a short one for most of the 256 compute units: 400 of 2560 107 -> 101, 480 of 3072 141 -> 133, 512 of
//    2048 112 -> 104 and 102 -> 95, of 4096 185 -> 168 and 174 -> 157; 320 of 2048 72 -> 72 and 80 -> 84, 384 of 2048 90 -> 84 and 85 -> 86; 560 of 1792
//    129 -> 129 and 112 -> 121, 640 of 2048 166 -> 165 and 146 -> 154, 704 of 2048 172 -> 166 and 152 -> 156;
//  * and again from three each on: 768 of 2000 177 -> 167 and 148 -> 145, of 4096 271 -> 262, 896 of 1792 181 -> 172 and 159 -> 157, 1024 of 4096 357 -> 341
//    and 332 -> 313.
// (4 -> 8 wavefronts, head dim 128, three streams, inputs from HBM; second figures: four query heads to a key head.  One stream gains as much or more, eight
// 1 to 4 %.)  Where batch times key heads is no multiple of 8, and workgroups therefore not placed by XCD, they are slower
// up to 512 workgroups (50 heads of 2048 109 -> 130, 25 of 4096 189 -> 207) and do not matter beyond.  Head dim 64 has too few pieces per block
// for 512 threads to stage.
bool wide_pays(long long tiles128, long long workgroups) {
  return tiles128 % 2 == 0 && tiles128 >= 14 && ((workgroups >= 400 && workgroups <= 512) || workgroups >= 768);
}

// Workgroups of 32 queries whose wavefronts share out the keys (hca_split_kernel; the same bits) pay
//  * where each gets a compute unit to itself, up to 256 of them: 16 heads of 64 on 4, 333 positions, two streams 9.8 -> 7.1 us, 4 heads of 128, 1500
//    positions, three streams 40.7 -> 25.8, 32 heads, 256 positions 10.8 -> 7.2; one key block (up to 64 positions) and no band has nothing to share out: 4.0 ->
//    4.1 and 4.9 -> 4.7, with a band 6.8 -> 5.2;
//  * in a second round of them only where the other kernel's chain is long: head dim 128 from 1000 positions on (512 workgroups of 1024 30.9 -> 24.9, of
//    2048 52.3 -> 39.6; 506 of 700 23.6 -> 22.7, of 333 13.1 -> 13.4 and 17.5 -> 16.2), 64, where a compute unit holds two, from 200 (448 of 200 7.2 ->
//    6.3 and 9.3 -> 6.9, 512 of 2048 32.9 -> 22.7; of 100 5.8 -> 5.8 and 7.9 -> 6.6);
//  * not beyond, where every 32 queries' own reads of keys and values fill the paths from the L2: 640 of 1024 positions 31.7 -> 35.3, 1024 of 2048 53.4 -> 77.9
//    (head dim 64 19.8 -> 20.0 and 33.5 -> 32.3, but 640 of 300 7.9 -> 9.6, of 700 15.3 -> 17.4).
// (three streams or one, inputs in the caches)
bool split_pays(int hd, int seq, int streams, long long workgroups) {
  if (workgroups <= 256) return seq > 64 || streams > 1;
  return workgroups <= 512 && seq >= (hd == 64 ? 200 : 1000);
}

template <int HD, int WAVES>
hipError_t launch_waves(const HcaArgs &a, hipStream_t st) {
  constexpr int kLds = HcaLds<HD, WAVES>::total;
  static bool lds_allowed[64] = {};
  const hipError_t e = allow_lds((const void *)hca_attention_kernel<HD, WAVES>, kLds, lds_allowed);
  if (e != hipSuccess) return e;
  const int G = a.hq / a.hkv;
  const int n_qt = (a.seq + WAVES * 32 - 1) / (WAVES * 32);
  const long long grid = (long long)a.batch * a.hkv * G * n_qt;
  if (grid > 0x7FFFFFFFll) return hipErrorInvalidValue;
  hipLaunchKernelGGL((hca_attention_kernel<HD, WAVES>), dim3((unsigned)grid), dim3(WAVES * 64), kLds, st, a);
  return hipGetLastError();
}

template <int HD>
hipError_t launch_split(const HcaArgs &a, hipStream_t st) {
  using L = SplitLds<HD>;
  static_assert(L::total(kMaxStreams) <= 160 * 1024, "the LDS of a compute unit");
  static bool lds_allowed[64] = {};
  const hipError_t e = allow_lds((const void *)hca_split_kernel<HD>, L::total(kMaxStreams), lds_allowed);
  if (e != hipSuccess) return e;
  const long long grid = (long long)a.batch * a.hq * ((a.seq + 31) / 32);
  if (grid > 0x7FFFFFFFll) return hipErrorInvalidValue;
  hipLaunchKernelGGL(hca_split_kernel<HD>, dim3((unsigned)grid), dim3(kSplitWaves * 64), L::total(a.n_streams), st, a);
  return hipGetLastError();
}

template <int HD>
hipError_t launch_hd(const HcaArgs &a, hipStream_t st) {
  if (split_pays(HD, a.seq, a.n_streams, (long long)a.batch * a.hq * ((a.seq + 31) / 32))) return launch_split<HD>(a, st);
  if constexpr (HD == 128) {
    const long long tiles = (a.seq + 127) / 128;
    if (wide_pays(tiles, (long long)a.batch * a.hq * ((tiles + 1) / 2))) return launch_waves<HD, 8>(a, st);
  }
  return launch_waves<HD, 4>(a, st);
}

}  // namespace

hipError_t launch_hca_attention(const HcaArgs &a, hipStream_t st) {
  if (a.n_streams < 1 || a.n_streams > kMaxStreams || a.batch < 1 || a.seq < 1 || a.hkv < 1 || a.hq < a.hkv || a.hq % a.hkv)
    return hipErrorInvalidValue;
  if (a.hd == 128) return launch_hd<128>(a, st);
  if (a.hd == 64) return launch_hd<64>(a, st);
  return hipErrorInvalidValue;
}

}  // namespace spec
