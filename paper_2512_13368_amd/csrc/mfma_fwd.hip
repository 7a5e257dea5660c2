// Fused forward on the matrix cores for bf16, d = 64, block size 32 (Eq. 1 under the two branch masks, Eq. 16-19), plus
// the same-style dense causal comparison.  Block size 64 is the four-wavefront kernel of mfma_fwd4.hip.
//
// One wavefront per (row, head, query block).  It stages its K and V tiles itself with direct global->LDS loads
// (16 bytes per lane, whole 128-byte rows per 8 lanes, XOR-swizzled so that the operand reads are bank-conflict
// free), so the tile loop has no barrier: the wavefront only waits for its own loads.
//
// Per tile it computes S^T = K Q^T with four v_mfma_f32_32x32x16_bf16 (keys are the M dimension, so every lane owns ONE
// query column and 16 of its logits; Q is pre-multiplied by scale*log2(e), rounded to bf16 once, so that the result is the
// base-2 exponent), takes the exponentials, and feeds P^T straight from the accumulator registers (converted to bf16) as the B
// operand of O^T += V^T P^T (four more MFMAs).  The key order inside a contraction slab is whatever the accumulator
// layout dictates; V^T is read from LDS with the transposing ds_read_b64_tr_b16 in exactly that order, so P never moves
// between lanes.  Row sums are plain fp32 adds: the packed dot-product instructions execute on the matrix pipeline
// and would stall the MFMAs.
//
// ONE WALK, NO REFERENCE.  Both branches see the same logits, so a tile that the two visit (the query block's own always, a
// window block whenever it is also selected) is loaded, multiplied and exponentiated once and masked twice.  The exponentials are
// those of the logits themselves, with no running maximum: while a row's sum stays within 2^+-60 (and its output finite)
// nothing has overflowed or been lost in fp32, and bf16 probabilities carry the same exponents.  A block with a row
// outside that range is walked again with the row maxima, found by a walk of their own, as references: with every block outside
// it (logits in the hundreds) the forward at B=128 H=4 L=1024, lengths U[100,1024] takes 176 us instead of 56.
// The walk starts with the block's own tile, whose place is known before anything has been read.
// A wavefront's life is latency (about ten tiles): at B=128 H=4 L=1024 k=8 w=64, lengths U[100,1024], two walks with online
// references took 91 us (saving: 139), this one 66 (110).
//
// Outputs leave through the wavefront's staging rows so that every store covers whole rows.
#include "launch.h"
#include "mfma_common.h"

namespace blossom {

using namespace mfma;

namespace {

constexpr int BLK = 32;
constexpr int TILE = BLK * D;    // bf16 elements of one staged tile (rows of 128 bytes, swizzled)
constexpr int kFewKeys = 32;     // rows seeing fewer keys than this get two-term bf16 probabilities
constexpr float kSumHi = 1.152921504606847e18f, kSumLo = 1.0f / kSumHi;  // 2^60: see ONE WALK above

// s_waitcnt immediate that waits until at most n vector-memory operations are outstanding and
// leaves the other counters alone (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt 6:4,
// lgkmcnt 11:8).
constexpr int vmcnt_imm(int n) { return (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); }
// The lane id, opaque to the compiler: what is derived from it is computed where it is used.
__device__ __forceinline__ int fresh_lane()
{
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}
constexpr int kLgkm0 = 15 | (7 << 4) | (3 << 14);  // lgkmcnt(0), the others at their maximum

}  // namespace

// EQ15: the short-term mask is all of Eq. 15 with mask block BLK, or (SUB) a power of two below it
// (compile-time, so that the plain causal window compiles to exactly the code it had without it)
template <bool EQ15, bool SUB>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3, 3))) void fwd_mfma_kernel(
    const uint16_t *__restrict__ Q, const uint16_t *__restrict__ K, const uint16_t *__restrict__ V,
    const int *__restrict__ valid_len, const int *__restrict__ sel, const float *__restrict__ gate_w,
    const float *__restrict__ gate_b, uint16_t *__restrict__ O, float *__restrict__ o_lt_out,
    float *__restrict__ o_st_out, float *__restrict__ lse_lt_out, float *__restrict__ lse_st_out, int dense,
    KParams p)
{
  __shared__ __attribute__((aligned(1024))) uint16_t Ks[TILE];
  __shared__ __attribute__((aligned(1024))) uint16_t Vs[TILE];
  __shared__ float gate_s[2 * D];  // this head's gate weights, fetched at the start, used at the very end

  const int lane = threadIdx.x;
  const int lq = lane & 31;  // query column (and key row of the K operand, d row of the V^T operand)
  const int lh = lane >> 5;  // which half of each 16-wide contraction slab
  const unsigned vid = xcd_spread(blockIdx.x, (unsigned)(p.B * p.H), (unsigned)p.nq);
  const int bh = (int)(vid / p.nq);
  const int I = p.NB - 1 - (int)(vid % p.nq);
  const int h = bh % p.H;
  const size_t head = (size_t)bh * p.L * D;
  const int qbase = I * BLK;
  const int iq = qbase + lq;

  // ---- staging: 32 rows (4 x 1 KB) of K or V per tile ----
  // LDS position of 16-byte chunk c of row r: r*128 + ((c ^ swz(r)) * 16), free of bank conflicts in both read patterns.
  // A tile's rows are contiguous in memory, and the LDS copy keeps the 128-byte row pitch, so
  // one uniform base (SGPRs) + one per-lane byte offset + the same immediate for the global
  // and the LDS side addresses all four 8-row slices.
  const char *Kh = reinterpret_cast<const char *>(K + head);
  const char *Vh = reinterpret_cast<const char *>(V + head);
  const int J_rag = p.L % BLK != 0 ? p.NB - 1 : -2;  // the one block whose rows run past the end, if any
  // (the lane's offset is rebuilt from the lane id at each use: registers are short)
  auto ld_offset = [&](int l) { return (unsigned)((l >> 3) * D + ((l & 7) ^ swz(l >> 3)) * 8) * 2u; };  // bytes; odd 8-row slices: ^ 32
  auto stage = [&](const char *src_head, uint16_t *dst_tile, int J) __attribute__((always_inline)) {
    const unsigned ld_lane = ld_offset(fresh_lane());
    J = J < 0 ? I : J;  // (block -1, whose exponentials are all masked: values that are certainly finite)
    const char *src = src_head + (size_t)J * (TILE * 2);  // uniform
    lds_void *dst = (lds_void *)dst_tile;
    if (J != J_rag) {
      const unsigned ld_odd = ld_lane ^ 32u;
      __builtin_amdgcn_global_load_lds((glb_void *)(src + ld_lane), dst, 16, 0, 0);
      __builtin_amdgcn_global_load_lds((glb_void *)(src + ld_odd), dst, 16, 1024, 0);
      __builtin_amdgcn_global_load_lds((glb_void *)(src + ld_lane), dst, 16, 2048, 0);
      __builtin_amdgcn_global_load_lds((glb_void *)(src + ld_odd), dst, 16, 3072, 0);
    } else {  // last, partial block: rows past the end are clamped (they are causally masked anyway)
      // (the empty asm hides that J is a constant here: the clamped per-lane offsets would
      // otherwise be computed ahead of the loop and held in registers throughout)
      asm volatile("" : "+s"(J));
      const int ld_row = fresh_lane() >> 3;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int over = max(0, J * BLK + ld_row + 8 * u - (p.L - 1));
        const unsigned off = ((u & 1) ? ld_lane ^ 32u : ld_lane) + (unsigned)((8 * u - over) * D * 2);
        __builtin_amdgcn_global_load_lds((glb_void *)(src + off), (lds_void *)(dst_tile + 8 * u * D), 16, 0, 0);
      }
    }
  };

  // (padding is not read: the valid length, a scalar load that mostly hits its cache, is waited for first)
  const int n = clamp_len(valid_len[bh / p.H], p.L);
  const int p0 = p.L - n;
  const bool q_ok = iq < p.L && iq >= p0;

  if (min((I + 1) * BLK, p.L) <= p0) {  // no valid query in the block: zero outputs
    zero_rows(O + head, qbase, 32, p.L, lane);
    if (o_lt_out) {
      zero_rows(o_lt_out + head, qbase, 32, p.L, lane);
      zero_rows(o_st_out + head, qbase, 32, p.L, lane);
    }
    if (iq < p.L && lh == 0) {
      if (lse_lt_out) lse_lt_out[(size_t)bh * p.L + iq] = 0.0f;
      if (lse_st_out) lse_st_out[(size_t)bh * p.L + iq] = 0.0f;
    }
    return;
  }

  // ---- everything else the prologue needs from memory is requested before anything is waited for ----
  const int *my_sel = dense ? nullptr : sel + ((size_t)bh * p.NB + I) * p.k;
  const int sel0 = (!dense && lane < p.k) ? my_sel[lane] : -1;  // first 64 entries of the selection row
  uint4 qraw[4];
  {
    const uint16_t *qrow = Q + head + (size_t)min(iq, p.L - 1) * D;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) qraw[kk] = *reinterpret_cast<const uint4 *>(qrow + 16 * kk + 8 * lh);
  }
  float gate_mine[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) gate_mine[c] = dense ? 0.0f : gate_w[(size_t)h * 2 * D + c * 64 + lane];
  stage(Kh, Ks, I);  // the walk's first tile
  stage(Vh, Vs, I);


  // ---- the short-term tiles: window blocks J_lo..I; with the full mask of Eq. 15 also the blocks I - 2^r below them,
  // r = r0 .. r0 + n_pow - 1.  The mask block is BLK or a power of two below it (`sub`): then the mask-block distances
  // 2^r below one tile reach into block I - 1, which joins the window range, the larger ones land on the same blocks I - 2^r'
  // (at the row's own offset), and every short-term tile is masked element by element with the three cases of Eq. 15. ----
  const int J_first = p0 / BLK;
  constexpr bool sub = EQ15 && SUB;  // (compile-time: the mask block = BLK variant keeps its code and registers)
  const int sub_sh = sub ? __builtin_ctz((unsigned)p.sblk) : 0;
  int J_lo = I, n_st = 0, n_win = 0, r0 = 0;  // (dense: none)
  if (!dense) {
    const int lowpos = I * BLK - (p.w - 1);
    J_lo = lowpos <= 0 ? 0 : lowpos / BLK;
    if (sub) J_lo = min(J_lo, I - 1);
    J_lo = max(J_lo, J_first);
    n_win = I - J_lo + 1;
    n_st = n_win;
    if (EQ15 && I > J_first) {
      const int d_win = I - J_lo;                                     // largest block distance inside the window range
      r0 = d_win == 0 ? 0 : 32 - __builtin_clz((unsigned)d_win);      // smallest r with 2^r > d_win
      const int r_max = 31 - __builtin_clz((unsigned)(I - J_first));  // largest r with I - 2^r >= J_first
      n_st += max(0, r_max - r0 + 1);
    }
  }
  // tile t of them, own block first
  auto st_tile = [&](int t) { return !EQ15 || t < n_win ? I - t : I - (1 << min(r0 + t - n_win, 30)); };

  // ---- the selection list, and which of its entries are short-term tiles too ----
  // Lane t: where the short-term tile t stands in the list (-1: nowhere).  Entries outside [0, NB) are skipped
  // wherever they stand: the walk runs up to the last valid one.
  int n_lt = 0, at = -1;
  bool lt_few = true;   // the selected past blocks hold fewer than kFewKeys valid keys
  bool lt_any = dense;  // the list names a block with a valid key up to the own one: every valid row sees a key of it
  const int n_look = min(n_st, 64);
  if (dense) {
    n_lt = I - J_first + 1;
  } else {
    for (int e0 = 0; e0 < p.k; e0 += 64) {
      const int e = e0 + lane;
      const int J = e0 == 0 ? sel0 : (e < p.k ? my_sel[e] : -1);
      const bool ok = J >= 0 && J < p.NB;
      const unsigned long long okm = __ballot(ok);
      if (okm != 0ull) n_lt = e0 + 64 - __builtin_clzll(okm);
      // a full earlier block already brings a whole block of keys; only a partial first block may not
      const int vcount = min((J + 1) * BLK, p.L) - max(J * BLK, p0);
      if (__ballot(ok && J < I && vcount >= kFewKeys) != 0ull) lt_few = false;
      if (__ballot(ok && J <= I && vcount > 0) != 0ull) lt_any = true;
      for (int t = 0; t < n_look; ++t) {
        const unsigned long long hit = __ballot(J == st_tile(t));
        if (hit != 0ull && lane == t && at < 0) at = e0 + __builtin_ctzll(hit);
      }
    }
  }
#pragma unroll
  for (int c = 0; c < 2; ++c) gate_s[c * 64 + lane] = gate_mine[c];

  // Q^T operand: lane (query lq, half lh) holds c*Q[iq][16*kk + 8*lh .. +7] for the 4 slabs kk,
  // c = scale*log2(e), rounded to bf16: the matrix cores then produce base-2 exponents directly.
  bf16x8 qf[4];
  auto scale_q = [&](const uint4 (&raw)[4]) __attribute__((always_inline)) {
    const float c2 = p.scale * kLog2e;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const uint32_t w[4] = {raw[kk].x, raw[kk].y, raw[kk].z, raw[kk].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        qf[kk][2 * e] = (__bf16)(bf_lo(w[e]) * c2);
        qf[kk][2 * e + 1] = (__bf16)(bf_hi(w[e]) * c2);
      }
    }
  };
  scale_q(qraw);
  __syncthreads();

  // ---- the walk: the short-term tiles that are selected too (the own block first), the other short-term ones (t < 64, then
  // any beyond, which are taken as such), the rest of the selection list (one scalar load per tile) ----
  const unsigned long long both_st = __ballot(at >= 0), only_st = __ballot(lane < n_look && at < 0);
  // the first list entry from e on that is not a short-term tile
  auto list_next = [&](int e) -> int {
    while (e < n_lt && !dense && __ballot(at == e) != 0ull) ++e;
    return e;
  };
  // its block; entries outside [0, NB) and blocks of nothing but padding, whose values may be anything, become -1, a tile that is skipped
  auto list_block = [&](int e) -> int {
    typedef const int __attribute__((address_space(4))) *const_int_ptr;  // read-only: loads become scalar
    const int J = __builtin_amdgcn_readfirstlane(dense ? J_first + e : ((const_int_ptr)my_sel)[e]);
    return J >= J_first && J < p.NB ? J : -1;
  };
  struct Place {  // what is still to be walked
    unsigned long long both, only;
    int far, e;
  };
  const Place start{both_st, only_st, 64, list_next(0)};
  auto left = [&](const Place &w) { return w.both != 0ull || w.only != 0ull || w.far < n_st || w.e < n_lt; };
  auto tile_at = [&](const Place &w) -> int {
    if (w.both != 0ull) return st_tile((int)__builtin_ctzll(w.both));
    if (w.only != 0ull) return st_tile((int)__builtin_ctzll(w.only));
    return w.far < n_st ? st_tile(w.far) : w.e < n_lt ? list_block(w.e) : -1;
  };

  // ---- per-lane LDS read offsets ----
  const int r16 = lane & 15;
  int koff = 2 * (lq * D + ((lh ^ swz(lq)) * 8));  // bytes; slab kk: ^ 32*kk
  const int v_row = 4 * lh + (r16 >> 2);             // the second read of an operand: 8 rows further down, another swizzle
  int voff = 2 * (v_row * D + (((2 * ((lane >> 4) & 1) + ((r16 & 3) >> 1)) ^ swz(v_row)) * 8) + 4 * (r16 & 1));  // bytes; channel half mb: ^ 64*mb

  // Rows that see only a few keys have large probabilities, and rounding those to bf16 would leave a relative error
  // of 2^-9 in the saved branch outputs, which backward amplifies through D = dO_x.o_x.  Blocks that may hold such rows
  // (fewer than kFewKeys keys) feed P to the matrix cores as a two-term bf16 sum (hi + lo); everyone else uses one term.
  const int hp_st = !dense && (p.w < kFewKeys || I * BLK - p0 + 1 < kFewKeys);
  const int hp_lt = dense ? I * BLK - p0 + 1 < kFewKeys : __builtin_amdgcn_readfirstlane((int)lt_few);

  // Zeroes the entries of `x` that the row does not see.
  // long-term: p0 <= key <= q; window: max(p0, q - w + 1) <= key <= q
  auto mask = [&](int J, bool short_term, f32x16 &x) __attribute__((always_inline)) {
    // (The query row is rebuilt from the lane id inside a volatile asm: everything derived
    // below would otherwise be loop invariant, get hoisted, and sit in registers or spill
    // slots across the whole walk.)
    const int ql = fresh_lane();
    const int q = qbase + (ql & 31);
    const int lh_ = ql >> 5;
    asm volatile("" : "+s"(J));
    // band-masked by the window, unless Eq. 15 shows the whole block (power-of-two block distance)
    const bool windowed = short_term && !(EQ15 && !sub && is_pow2(I - J));
    int wlo = q - p.w + 1;
    if (EQ15 && q >= p.last_lo) wlo = min(wlo, p.last_lo);  // third case of Eq. 15: the last block is visible to its own rows
    const int lo = windowed ? max(p0, wlo) : p0;
    if (EQ15 && sub && windowed && J < J_lo && J * BLK >= p0) {
      // A block I - 2^r' below the window range, all of it valid: no key of it lies in a window or in
      // the last block, and a mask-block distance 2^r' * (BLK / blk) + delta with |delta| < BLK / blk <=
      // half of it is a power of two only for delta = 0: row and key share the mask block within their tiles.
      const int qo = q & (BLK - 1);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int ko = 4 * lh_ + 8 * (i >> 2) + (i & 3);
        x[i] = (((qo ^ ko) >> sub_sh) == 0 && q >= p0) ? x[i] : 0.0f;
      }
      return;
    }
    if (EQ15 && sub && windowed) {
      // window range as above, or (valid, causal and) a power-of-two mask-block distance, or a last-block key
      const int base = J * BLK + 4 * lh_;
      const unsigned span = (unsigned)(q - lo);  // wraps to huge when q < lo: handled by `any`
      const bool any = q >= lo;
      const unsigned cspan = (unsigned)(q - p0);
      const bool cany = q >= p0;
      const int qmb = q >> sub_sh;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int key = base + 8 * (i >> 2) + (i & 3);
        const int d = qmb - (key >> sub_sh);
        const bool far = cany & ((unsigned)(key - p0) <= cspan) & ((d > 0 && (d & (d - 1)) == 0) | (key >= p.last_lo));
        const bool vis = (any & ((unsigned)(key - lo) <= span)) | far;
        x[i] = vis ? x[i] : 0.0f;
      }
      return;
    }
    keep_rows(x, row_bits(lo - J * BLK, q - J * BLK), lh_);
  };
  // does every row of the block see the whole tile? (uniform)
  auto whole_lt = [&](int J) { return J < I && J * BLK >= p0; };
  auto whole_st = [&](int J) {
    return J < I && J * BLK >= p0 && (EQ15 ? !sub && is_pow2(I - J) : J * BLK >= qbase + 31 - p.w + 1);
  };

  f32x16 o_lt[2], o_st[2];  // [channel half]
  float l_lt, l_st;         // this lane's parts of the row sums
  auto clear = [&]() {
    l_lt = l_st = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; ++i) o_lt[0][i] = o_lt[1][i] = o_st[0][i] = o_st[1][i] = 0.0f;
  };
  auto read_k = [&](bf16x8 (&kf)[4]) __attribute__((always_inline)) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) kf[kk] = *reinterpret_cast<const bf16x8 *>(reinterpret_cast<const char *>(Ks) + (koff ^ 32 * kk));
  };
  // V^T operands: [t][mb], keys in accumulator order
  auto read_v = [&](bf16x8 (&vf)[2][2]) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int mb = 0; mb < 2; ++mb) {
        const char *a0 = reinterpret_cast<const char *>(Vs) + 32 * t * D + (voff ^ 64 * mb);
        const char *a8 = reinterpret_cast<const char *>(Vs) + 32 * t * D + 16 * D + (voff ^ 64 * mb ^ 32);
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(a0));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)a8);
        vf[t][mb] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      }
  };
  auto logits = [&](const bf16x8 (&kf)[4]) __attribute__((always_inline)) -> f32x16 {
    f32x16 s = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk], qf[kk], s, 0, 0, 0);
    return s;
  };
  // o += V^T P, l += the lane's sum of P; hp: P as a two-term bf16 sum
  auto add = [&](const bf16x8 (&vf)[2][2], const f32x16 &P, auto hp, f32x16 (&o)[2], float &l) __attribute__((always_inline)) {
    bf16x8 pf[2];
    float sum_a = 0.0f, sum_b = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; i += 2) {
      pf[i >> 3][i & 7] = (__bf16)P[i];
      pf[i >> 3][(i & 7) + 1] = (__bf16)P[i + 1];
      sum_a += P[i];
      sum_b += P[i + 1];
    }
    l += sum_a + sum_b;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int mb = 0; mb < 2; ++mb) o[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[t][mb], pf[t], o[mb], 0, 0, 0);
    if (hp) {
      bf16x8 pl[2];
#pragma unroll
      for (int i = 0; i < 16; ++i) pl[i >> 3][i & 7] = (__bf16)(P[i] - (float)pf[i >> 3][i & 7]);
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) o[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[t][mb], pl[t], o[mb], 0, 0, 0);
    }
  };

  // ---- a step: its K goes to registers, then its V, which frees their buffers for the next tile's, on the way under this
  // one's work ----
  bf16x8 vf[2][2];
  auto step = [&](bool more, int J_nxt) __attribute__((always_inline)) -> f32x16 {  // the tile's exponentials, V in vf
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    asm volatile("" : "+v"(koff), "+v"(voff));
    bf16x8 kf[4];
    read_k(kf);
    __builtin_amdgcn_s_waitcnt(kLgkm0);
    if (more) stage(Kh, Ks, J_nxt);
    f32x16 s = logits(kf);
    read_v(vf);
    __builtin_amdgcn_s_waitcnt(kLgkm0);
    if (more) stage(Vh, Vs, J_nxt);
    return s;
  };
  auto to_exp = [&](f32x16 &s) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = __builtin_amdgcn_exp2f(s[i]);
  };
  clear();
  if (tile_at(start) != I) {  // (the own block is not selected, or dense)
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    stage(Kh, Ks, tile_at(start));
    stage(Vh, Vs, tile_at(start));
  }
  // (straight-line loops per kind of tile: accumulators updated under a condition are copied at every join)
  auto walk = [&](auto hp) __attribute__((always_inline)) {
    Place w = start;
    int J = tile_at(w);
#pragma unroll 1
    while (w.both != 0ull) {
      w.both &= w.both - 1;
      const int J_nxt = tile_at(w);
      f32x16 s = step(left(w), J_nxt), x;
      to_exp(s);
      x = s;
      if (!whole_lt(J)) mask(J, false, x);
      add(vf, x, hp, o_lt, l_lt);
      if (!whole_st(J)) mask(J, true, s);
      add(vf, s, hp, o_st, l_st);
      J = J_nxt;
    }
#pragma unroll 1
    while (w.only != 0ull || w.far < n_st) {
      if (w.only != 0ull) w.only &= w.only - 1;
      else ++w.far;
      const int J_nxt = tile_at(w);
      f32x16 s = step(left(w), J_nxt);
      to_exp(s);
      if (!whole_st(J)) mask(J, true, s);
      add(vf, s, hp, o_st, l_st);
      J = J_nxt;
    }
#pragma unroll 1
    while (w.e < n_lt) {
      w.e = list_next(w.e + 1);
      const bool more = w.e < n_lt;
      const int J_nxt = more ? list_block(w.e) : -1;
      f32x16 s = step(more, J_nxt);
      to_exp(s);
      if (!whole_lt(J)) mask(J, false, s);  // (all of a tile -1)
      add(vf, s, hp, o_lt, l_lt);
      J = J_nxt;
    }
  };
  if (hp_st | hp_lt) walk(std::true_type{});
  else walk(std::false_type{});

  // ---- closing: normalised outputs, lse, gate (Eq. 18-19) ----
  float ref_lt = 0.0f, ref_st = 0.0f, lse_lt, lse_st, inv_lt, inv_st, z;
  auto close = [&](float l, float ref, float &inv, float &lse) __attribute__((always_inline)) -> bool {
    l += __shfl_xor(l, 32);
    const bool ok = q_ok && l > 0.0f;
    inv = ok ? 1.0f / l : 0.0f;
    lse = ok ? (ref + __log2f(l)) * kLn2 : 0.0f;
    return l >= kSumLo && l <= kSumHi;
  };
  auto finish = [&]() __attribute__((always_inline)) -> bool {  // returns whether every row stayed in range
    bool good = close(l_lt, ref_lt, inv_lt, lse_lt) || !lt_any;  // (no key: zeros, and nothing to walk for)
    if (!dense) good = close(l_st, ref_st, inv_st, lse_st) && good;
    else inv_st = 0.0f;
    float z_lt = 0.0f, z_st = 0.0f;
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int d0 = 32 * mb + 8 * g + 4 * lh;
        float a[4], b[4];
        load4(gate_s + d0, a);
        load4(gate_s + D + d0, b);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          z_lt = fmaf(a[c], o_lt[mb][4 * g + c], z_lt);
          z_st = fmaf(b[c], o_st[mb][4 * g + c], z_st);
        }
      }
    z = z_lt * inv_lt + z_st * inv_st;
    z += __shfl_xor(z, 32);
    // (an output that is not finite, with a zero weight too, makes z not finite)
    return !q_ok || (good && fabsf(z) <= 3.0e38f);
  };
  if (__any(!finish())) {
    // A row left the range (or its output fp32's): each branch is walked again, first for its row maxima, then against them.
    // (Q is read again, so that it does not stay in registers from the first walk to here.)
    {
      const int el = fresh_lane();
      const uint16_t *qrow = Q + head + (size_t)min(qbase + (el & 31), p.L - 1) * D;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) qraw[kk] = *reinterpret_cast<const uint4 *>(qrow + 16 * kk + 8 * (el >> 5));
      scale_q(qraw);
    }
    auto each_tile = [&](bool short_term, auto &&f) __attribute__((always_inline)) {
      Place w = start;
#pragma unroll 1
      while (left(w)) {
        const int J = tile_at(w);
        const bool st = w.both != 0ull || w.only != 0ull || w.far < n_st, lt = w.both != 0ull || !st;
        if (w.both != 0ull) w.both &= w.both - 1;
        else if (w.only != 0ull) w.only &= w.only - 1;
        else if (w.far < n_st) ++w.far;
        else w.e = list_next(w.e + 1);
        if (J < 0 || !(short_term ? st : lt)) continue;
        stage(Kh, Ks, J);
        stage(Vh, Vs, J);
        f32x16 s = step(false, 0);
        f(J, s);
      }
    };
    auto again = [&](bool short_term, f32x16 (&o)[2], float &l, float &ref) __attribute__((always_inline)) {
      float top = kNegInf;
      each_tile(short_term, [&](int J, f32x16 &s) __attribute__((always_inline)) {
        f32x16 seen;
#pragma unroll
        for (int i = 0; i < 16; ++i) seen[i] = 1.0f;
        mask(J, short_term, seen);
#pragma unroll
        for (int i = 0; i < 16; ++i) top = fmaxf(top, seen[i] != 0.0f ? s[i] : kNegInf);
      });
      top = fmaxf(top, __shfl_xor(top, 32));
      ref = top == kNegInf ? 0.0f : top;
      l = 0.0f;
#pragma unroll
      for (int i = 0; i < 16; ++i) o[0][i] = o[1][i] = 0.0f;
      each_tile(short_term, [&](int J, f32x16 &s) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = __builtin_amdgcn_exp2f(s[i] - ref);
        mask(J, short_term, s);
        add(vf, s, std::true_type{}, o, l);
      });
    };
    again(false, o_lt, l_lt, ref_lt);
    if (!dense) again(true, o_st, l_st, ref_st);
    (void)finish();
  }

  // ---- stores ----
  // A lane holds 4 consecutive channels of ONE row per accumulator quad; stored directly, an
  // instruction would touch 32 rows with 16 or 32 bytes each.  The tiles go through this
  // wavefront's staging rows instead (free now, XOR-swizzled against bank conflicts) and leave
  // as whole rows: 256 contiguous bytes per 16 lanes (fp32), 128 per 8 lanes (bf16).
  const int row0 = qbase;  // first of the 32 rows
  int el = lane;  // opaque copy: keeps the store addressing out of the registers of the tile loop
  asm volatile("" : "+v"(el));
  const int elq = el & 31, elh = el >> 5;
  auto store_f32_rows = [&](float *dst, const f32x16 (&acc)[2], float by, uint16_t *piece_a, uint16_t *piece_b)
                            __attribute__((always_inline)) {
    float *pa = reinterpret_cast<float *>(piece_a);  // rows 0..15, 256 bytes each
    float *pb = reinterpret_cast<float *>(piece_b);  // rows 16..31
    float *mine = elq < 16 ? pa : pb;
    const int rl = elq & 15;
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int chunk = 8 * mb + 2 * g + elh;  // 16-byte chunk of the row
        *reinterpret_cast<float4 *>(mine + rl * 64 + ((chunk ^ rl) * 4)) =
            make_float4(acc[mb][4 * g] * by, acc[mb][4 * g + 1] * by, acc[mb][4 * g + 2] * by, acc[mb][4 * g + 3] * by);
      }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int rr = 4 * (i & 3) + (el >> 4), c = el & 15;
      const float4 v = *reinterpret_cast<const float4 *>((i < 4 ? pa : pb) + rr * 64 + ((c ^ rr) * 4));
      const int grow = row0 + 16 * (i >> 2) + rr;
      typedef float f32x4_t __attribute__((ext_vector_type(4)));
      const f32x4_t vv = {v.x, v.y, v.z, v.w};
      if (grow < p.L) __builtin_nontemporal_store(vv, reinterpret_cast<f32x4_t *>(dst + head + (size_t)grow * D + 4 * c));
    }
  };
  // o4(mb, g, e): the value of channel 32*mb + 8*g + 4*lh + e of this lane's row
  auto store_bf16_rows = [&](uint16_t *dst, auto o4, uint16_t *piece) __attribute__((always_inline)) {
    uint16_t *pt = piece;  // 32 rows of 128 bytes
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        uint2 pk;
        pk.x = pack2_bf16(o4(mb, g, 0), o4(mb, g, 1));
        pk.y = pack2_bf16(o4(mb, g, 2), o4(mb, g, 3));
        const int chunk = 4 * mb + g;  // 16-byte chunk (8 channels); this lane fills half lh of it
        *reinterpret_cast<uint2 *>(pt + elq * D + ((chunk ^ (elq & 7)) * 8) + 4 * elh) = pk;
      }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int rr = 8 * i + (el >> 3), c = el & 7;
      const uint4 v = *reinterpret_cast<const uint4 *>(pt + rr * D + ((c ^ (rr & 7)) * 8));
      const int grow = row0 + rr;
      if (grow < p.L) *reinterpret_cast<uint4 *>(dst + head + (size_t)grow * D + 8 * c) = v;
    }
  };
  const size_t lrow = (size_t)bh * p.L + iq;
  if (dense) {
    store_bf16_rows(O, [&](int mb, int g, int c) { return inv_lt * o_lt[mb][4 * g + c]; }, Ks);
    if (iq < p.L && lh == 0 && lse_lt_out) lse_lt_out[lrow] = lse_lt;
    return;
  }
  z += gate_b ? gate_b[h] : 0.0f;
  const float alpha = q_ok ? 1.0f / (1.0f + __expf(-z)) : 0.0f;
  const float by_lt = alpha * inv_lt, by_st = (1.0f - alpha) * inv_st;
  if (o_lt_out) {
    store_f32_rows(o_lt_out, o_lt, inv_lt, Ks, Vs);
    store_f32_rows(o_st_out, o_st, inv_st, Ks, Vs);
  }
  store_bf16_rows(O, [&](int mb, int g, int c) {
    return by_lt * o_lt[mb][4 * g + c] + by_st * o_st[mb][4 * g + c];
  }, Ks);
  if (iq < p.L && lh == 0) {
    if (lse_lt_out) lse_lt_out[lrow] = lse_lt;
    if (lse_st_out) lse_st_out[lrow] = lse_st;
  }
}

bool fwd_mfma_supported(const KParams &p, int dtype)
{
  return dtype == 1 && p.d == 64 && (p.b == 32 || p.b == 64) && !p.bidir &&
         (p.sblk == 0 || (is_pow2(p.sblk) && p.sblk <= p.b));
}

void launch_fwd_mfma(const KParams &p, const FwdArgs &a, hipStream_t st)
{
  if (p.b == 64) {
    launch_fwd_mfma4(p, a, st);
    return;
  }
  // (The last block alone goes through the same walk as among all blocks: a history's served outputs are those of its full run, bit for bit,
  // in a batch of any size.  Four wavefronts with every fourth tile each would take 51.4 instead of 59.1 us with the selection at B=16 H=8 L=8192
  // k=16 w=128, but add in another order.)
  const unsigned grid = (unsigned)(p.B * p.H * p.nq);
  auto u16 = [](const void *x) { return reinterpret_cast<const uint16_t *>(x); };
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(64), 0, st, u16(a.Q), u16(a.K), u16(a.V), a.valid_len, a.sel,
                       a.gate_w, a.gate_b, (uint16_t *)a.O, (float *)a.o_lt, (float *)a.o_st, a.lse_lt, a.lse_st,
                       a.dense, p);
  };
  const bool eq15 = p.sblk != 0 && !a.dense;
  const bool sub = eq15 && p.sblk < p.b;  // mask block smaller than the tile
  if (sub) go(fwd_mfma_kernel<true, true>);
  else if (eq15) go(fwd_mfma_kernel<true, false>);
  else go(fwd_mfma_kernel<false, false>);
}

}  // namespace blossom
