// Forward and backward on the fp32 matrix instructions for short sequences (Eq. 1 under the two branch
// masks, Eq. 16-19 and their chain rule, and the same-style dense causal comparison): fp32 or bf16
// storage, d in {8, 16, 32}, block size 8 or 16, sequences whose streamed tensors fit the LDS of a
// workgroup.  That is the paper's own regime (Sec. 4.1, Appendix E: histories of at most 200 items,
// hidden size 64 over 2 to 8 heads, selection block 16); the 64 x 64 bf16 tiles of the long-sequence
// kernels would be mostly padding there.
//
// One workgroup per (row, head), or per (row, key/value group) in the per-position form.  Positions are
// cut into 16-row tiles of v_mfma_f32_16x16x4_f32 (true fp32 products accumulated in fp32) whatever the
// block size; a selection block of 8 is half a tile and the selection is tested per element.  The tensors
// that a walk streams are staged once, as fp32, from the first valid tile on, into LDS rows of d + 4 floats
// (both operand read patterns below are then bank-conflict free); each wavefront walks whole tiles of its
// own with no barrier and no staging inside the walks.
//
// BOTH BRANCHES IN ONE WALK.  The branches share the logits, so a walk visits the union of the two tile
// sets once and applies two masks to one product: forward forms S once and adds P_lt V and P_st V;
// backward needs S, dO V^T, and, because dS = dS_lt + dS_st multiplies the same K and Q, one product each
// for dQ, dK and dV (dV: the coefficient of dO is a_lt P_lt + a_st P_st, the gate part is a rank-one term
// per key).  Which tiles a walk visits comes from bit masks over tiles (one pair of 64-bit words per query
// tile and per key tile), built once per workgroup from the selection rows and the mask geometry.
//   forward: S^T = K Q^T, keys as the M dimension: lane (q = lane % 16, g = lane / 16) owns query column
//            q and the logits of keys 4g .. 4g+3 of the tile; O^T += V^T P^T with P^T = the accumulator of
//            S^T as it stands (step r contracts key 4g + r of every lane group).
//   dQ:      same orientation: S^T and G_x^T = V dO_x^T leave the matrix cores in the layout in which
//            dS^T is the B operand of dQ^T += K^T dS^T.
//   dK/dV:   queries as the M dimension (lane (key, g): key column, query rows 4g .. 4g+3); the per-row
//            constants are 16-byte broadcast reads from LDS, the lane's own K and V rows are registers.
// A contraction over channels takes channel (d/4)*g + s in step s, so that a lane's operands are d/4
// consecutive floats: one or two 16-byte LDS reads per tile instead of d/4 reads.
//
// EXPONENTIALS WITHOUT A RUNNING MAXIMUM.  |logit| <= |q| |k|: where the largest such bound of a query tile is
// at most 60 (in log2 units) exp2 of the logits themselves neither overflows nor loses accuracy in fp32, so
// neither a maximum nor a rescale is needed and the branches share one exponential.  Otherwise the walk runs
// once more beforehand for the two row maxima.
//
// Backward is one kernel: per-row gate pass (alpha, dz, D_x and the gate-weight gradients of its (row, head)),
// dK/dV, then dQ; K, V, Q, dO, o_lt and o_st come from memory once.  With dO_x = a_x*dO + dz*Wg_x the upstream
// gradient of branch x (a_lt = alpha, a_st = 1 - alpha) and D_x = dO_x.o_x:
//   P_ij = exp(scale*q_i.k_j - lse_x,i),  dS_ij = P_ij * (dO_x,i.v_j - D_x,i),
//   dQ_i = scale * sum_j dS_ij k_j,  dK_j = scale * sum_i dS_ij q_i,  dV_j = sum_i P_ij dO_x,i.
// Masks (the causal window, or all of Eq. 15 in its causal or its bidirectional form), gate, outputs and padding
// rules are those of the scalar kernels of generic.hip; shapes outside this range stay there.
#include "launch.h"

namespace blossom {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr float kLog2eF = 1.4426950408889634f;
constexpr float kLn2F = 0.6931471805599453f;
constexpr float kNegInfF = -__builtin_huge_valf();
constexpr float kHugeF = 1.0e30f;
constexpr size_t kResLdsMax = 160 * 1024;
constexpr int kTile = 16;
constexpr int kMaxTiles = 64;        // tile masks are 64-bit words
constexpr float kSmallLogit = 60.0f;  // log2 units: exp2 of such a logit, and sums over a row, stay far inside fp32

template <int D>
struct Geo {
  static constexpr int CPL = D / 4;            // channels per lane of a channel contraction: CPL*g .. CPL*g + CPL-1
  static constexpr int NMB = (D + 15) / 16;    // 16-channel output blocks (d = 8 fills half of one)
  static constexpr int LDR = D + 4;            // floats per staged row (12, 20 or 36: conflict free, 16-byte rows)
};

// CPL consecutive elements as floats
template <int N>
__device__ __forceinline__ void load_n(const float *p, float (&o)[N])
{
  if constexpr (N == 2) {
    const float2 v = *reinterpret_cast<const float2 *>(p);
    o[0] = v.x; o[1] = v.y;
  } else {
#pragma unroll
    for (int i = 0; i < N; i += 4) {
      const float4 v = *reinterpret_cast<const float4 *>(p + i);
      o[i] = v.x; o[i + 1] = v.y; o[i + 2] = v.z; o[i + 3] = v.w;
    }
  }
}
template <int N>
__device__ __forceinline__ void load_n(const bf16_t *p, float (&o)[N])
{
  if constexpr (N == 2) {
    const uint32_t v = *reinterpret_cast<const uint32_t *>(p);
    o[0] = __uint_as_float(v << 16);
    o[1] = __uint_as_float(v & 0xFFFF0000u);
  } else if constexpr (N == 4) {
    load4(p, o);
  } else {
    const uint4 v = *reinterpret_cast<const uint4 *>(p);
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o[2 * i] = __uint_as_float(w[i] << 16);
      o[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
    }
  }
}
template <int N>
__device__ __forceinline__ void store_n(float *p, const float (&o)[N])
{
  if constexpr (N == 2) {
    *reinterpret_cast<float2 *>(p) = make_float2(o[0], o[1]);
  } else {
#pragma unroll
    for (int i = 0; i < N; i += 4) *reinterpret_cast<float4 *>(p + i) = make_float4(o[i], o[i + 1], o[i + 2], o[i + 3]);
  }
}
template <int N>
__device__ __forceinline__ void zero_n(float (&o)[N])
{
#pragma unroll
  for (int i = 0; i < N; ++i) o[i] = 0.0f;
}
template <int N>
__device__ __forceinline__ float dot_n(const float (&a)[N], const float (&b)[N], float c)
{
#pragma unroll
  for (int i = 0; i < N; ++i) c = fmaf(a[i], b[i], c);
  return c;
}
// sum over the four lane groups of a column
__device__ __forceinline__ float sum_g(float x)
{
  x += __shfl_xor(x, 16);
  return x + __shfl_xor(x, 32);
}

// A operand of a product whose contraction runs over the 16 rows of a staged tile: element r is row 4g + r,
// column `col` (d = 8: columns 8..15 hold anything, their output rows are never stored)
template <int LDR>
__device__ __forceinline__ void col_frag(const float *tile, int g, int col, float (&o)[4])
{
  const float *p = tile + 4 * g * LDR + col;
#pragma unroll
  for (int r = 0; r < 4; ++r) o[r] = p[r * LDR];
}

// lane (col, g) holds channels 16*mb + 4g + r of one row in a[mb][r]: stores those below D
template <typename T, int D>
__device__ __forceinline__ void store_row4(T *dst_row, const f32x4 (&a)[Geo<D>::NMB], int g)
{
#pragma unroll
  for (int mb = 0; mb < Geo<D>::NMB; ++mb)
    if (16 * mb + 4 * g < D) {
      const float v[4] = {a[mb][0], a[mb][1], a[mb][2], a[mb][3]};
      store4(dst_row + 16 * mb + 4 * g, v);
    }
}

// the same for a gradient row: scaled (zeros where the row is not kept), rotated back when the caller's rows
// went through the rotary embedding (four consecutive channels = two channel pairs)
template <typename T, int D>
__device__ __forceinline__ void store_grad_row(T *dst_row, const f32x4 (&a)[Geo<D>::NMB], float scale, bool keep,
                                               const KParams &p, bool unrope, int pos, int g)
{
#pragma unroll
  for (int mb = 0; mb < Geo<D>::NMB; ++mb)
    if (16 * mb + 4 * g < D) {
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = keep ? a[mb][e] * scale : 0.0f;
      if (unrope && p.rope_cos != nullptr) {
        const int pair = 8 * mb + 2 * g;
        unrope_pair(p, pos, pair, D / 2, v[0], v[1]);
        unrope_pair(p, pos, pair + 1, D / 2, v[2], v[3]);
      }
      store4(dst_row + 16 * mb + 4 * g, v);
    }
}

// zeros for the `count` elements from dst on (whole rows: a multiple of 8 elements, 16-byte aligned)
template <typename T>
__device__ __forceinline__ void zero_fill(T *dst, int count, int tid, int nthr)
{
  uint4 *q = reinterpret_cast<uint4 *>(dst);
  const int pieces = count * (int)sizeof(T) / 16;
  for (int i = tid; i < pieces; i += nthr) q[i] = make_uint4(0u, 0u, 0u, 0u);
}

// ---- what a workgroup knows about its masks -----------------------------------------------------------------
// In LDS, as 32-bit words:
//   tm_lt, tm_st [NT][2]   bit T: query tile I walks key tile T in the branch
//   cm_lt, cm_st [NT][2]   bit I: key tile T is walked by query tile I            (backward)
//   selw [NW][SR]          selection bits: word w of row x, bit e: key block 32*w + e is selected; x is a query block,
//                          or a position in the per-position form
//   kid [16*NT]            mask block of each position (Eq. 15)
struct MaskLayout {
  int NT, NW, SR;
  int tm_lt, tm_st, cm_lt, cm_st, selw, kid, words;
};
__host__ __device__ inline MaskLayout mask_layout(const KParams &p, bool perpos, bool bwd)
{
  MaskLayout m;
  m.NT = (p.L + kTile - 1) / kTile;
  m.NW = (p.NB + 31) / 32;
  m.SR = perpos ? kTile * m.NT : 2 * m.NT;
  int o = 0;
  m.tm_lt = o; o += 2 * m.NT;
  m.tm_st = o; o += 2 * m.NT;
  m.cm_lt = o; o += bwd ? 2 * m.NT : 0;
  m.cm_st = o; o += bwd ? 2 * m.NT : 0;
  m.selw = o; o += m.NW * m.SR;
  o = (o + 3) / 4 * 4;
  m.kid = o; o += p.sblk > 0 ? kTile * m.NT : 0;
  m.words = (o + 3) / 4 * 4;
  return m;
}

__device__ __forceinline__ unsigned long long tile_mask(const unsigned *m, int off, int I)
{
  const unsigned lo = __builtin_amdgcn_readfirstlane(m[off + 2 * I]);
  const unsigned hi = __builtin_amdgcn_readfirstlane(m[off + 2 * I + 1]);
  return ((unsigned long long)hi << 32) | lo;
}

// Fills the mask words (the caller synchronises afterwards).  bh_sel: the (row, head) or (row, group) index of the
// selection rows; sel == nullptr: dense causal attention, every tile up to the own one in the long-term masks.
template <int BK, bool PERPOS, bool BWD>
__device__ __forceinline__ void build_masks(unsigned *m, const MaskLayout &ml, const KParams &p, const int *sel, int bh_sel,
                                            int p0, int tid, int nthr)
{
  const int NT = ml.NT;
  for (int i = tid; i < ml.kid; i += nthr) m[i] = 0u;
  if (p.sblk > 0)
    for (int i = tid; i < kTile * NT; i += nthr) reinterpret_cast<int *>(m)[ml.kid + i] = i / p.sblk;
  __syncthreads();
  const int T0 = p0 / kTile;
  auto set_tile = [&](int tm, int cm, int I, int J) {
    atomicOr(&m[tm + 2 * I + (J >> 5)], 1u << (J & 31));
    if (BWD) atomicOr(&m[cm + 2 * J + (I >> 5)], 1u << (I & 31));
  };
  // short-term reach of every pair of tiles
  const int *kid = reinterpret_cast<const int *>(m) + ml.kid;
  for (int idx = tid; idx < NT * NT; idx += nthr) {
    const int I = idx / NT, J = idx - I * NT;
    if (J < T0 || I < T0 || (J > I && !p.bidir)) continue;
    if (!sel) {
      set_tile(ml.tm_lt, ml.cm_lt, I, J);
      continue;
    }
    const int dist = (I > J ? I - J : J - I) * kTile - (kTile - 1);  // smallest distance of the two tiles' positions
    bool reach = dist < p.w;
    if (!reach && p.sblk > 0) {
      const int q_lo = kid[I * kTile], q_hi = kid[min(I * kTile + kTile - 1, p.L - 1)];
      const int k_lo = kid[J * kTile], k_hi = kid[min(J * kTile + kTile - 1, p.L - 1)];
      reach = min(J * kTile + kTile - 1, p.L - 1) >= p.last_lo ||
              (J <= I ? holds_pow2(q_lo - k_hi, q_hi - k_lo) : holds_pow2(k_lo - q_hi, k_hi - q_lo));
    }
    if (reach) set_tile(ml.tm_st, ml.cm_st, I, J);
  }
  if (!sel) return;
  // selection rows (entries outside [0, NB), blocks after the query and blocks without a valid key drop out)
  const int rows = PERPOS ? p.L : p.NB;
  const int *s = sel + (size_t)bh_sel * rows * p.k;
  for (int idx = tid; idx < rows * p.k; idx += nthr) {
    const int x = idx / p.k;
    const int J = s[idx];
    const int I = PERPOS ? x / kTile : x * BK / kTile;
    const int q_hi = PERPOS ? x : x * BK + BK - 1;  // last position of the row or block
    if (J < 0 || J >= p.NB || q_hi < p0 || (J * BK > q_hi && !p.bidir) || (J + 1) * BK <= p0) continue;
    atomicOr(&m[ml.selw + (J >> 5) * ml.SR + x], 1u << (J & 31));
    set_tile(ml.tm_lt, ml.cm_lt, I, J * BK / kTile);
  }
}

// short-term visibility of a (query, key) pair that the causal and validity tests have let through
__device__ __forceinline__ bool st_sees(const KParams &p, int diff, int kid_diff, int key)
{
  if (p.bidir) {
    diff = abs(diff);
    kid_diff = abs(kid_diff);
  }
  bool v = diff < p.w;
  if (p.sblk > 0) v = v || (kid_diff > 0 && (kid_diff & (kid_diff - 1)) == 0) || key >= p.last_lo;
  return v;
}

}  // namespace

// =============================================================================================
// forward
// =============================================================================================
// PERPOS: the long-term branch takes one selection row per query POSITION and key/value group (the
// selection rule as printed, Eq. 8-13 with Eq. 4-5): K and V are [B,G,L,d], `sel` is [B,G,L,k] with
// selection blocks of BK positions.  A workgroup serves the hpg query heads of its group, which share its
// staged keys and values (hpg = 1 otherwise).
template <typename T, int D, int BK, bool PERPOS>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) void fwd_res_kernel(
    const T *__restrict__ Q, const T *__restrict__ K, const T *__restrict__ V, const int *__restrict__ valid_len,
    const int *__restrict__ sel, const float *__restrict__ gate_w, const float *__restrict__ gate_b,
    T *__restrict__ O, float *__restrict__ o_lt_out, float *__restrict__ o_st_out, float *__restrict__ lse_lt_out,
    float *__restrict__ lse_st_out, int hpg, KParams p)
{
  constexpr int CPL = Geo<D>::CPL, NMB = Geo<D>::NMB, LDR = Geo<D>::LDR;
  extern __shared__ __attribute__((aligned(16))) float lds_res[];
  __shared__ float red_s[16];
  const MaskLayout ml = mask_layout(p, PERPOS, false);
  const int NT = ml.NT;
  float *Ks = lds_res;
  float *Vs = Ks + NT * kTile * LDR;
  unsigned *mw = reinterpret_cast<unsigned *>(Vs + NT * kTile * LDR + 16);

  const int tid = threadIdx.x, nthr = blockDim.x;
  const int lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), W = nthr >> 6;
  const int bg = blockIdx.x;  // (row, key/value head)
  const int G = p.H / hpg;
  const int b = bg / G;
  const int n = clamp_len(valid_len[b], p.L);
  const int p0 = p.L - n;
  const int T0 = p0 / kTile;
  const int q = lane & 15, g = lane >> 4;
  const size_t head_kv = (size_t)bg * p.L * D;
  const bool dense = sel == nullptr;
  const int row_lo = (p.NB - p.nq) * BK;  // first row that is written (serving mode: the last block's)

  if (n == 0 || T0 * kTile > row_lo) {  // rows before the first valid tile: outputs are zero
    for (int hh = 0; hh < hpg; ++hh) {
      const size_t r0 = (size_t)(bg * hpg + hh) * p.L + row_lo;
      const int rows = (n == 0 ? p.L : T0 * kTile) - row_lo;
      zero_fill(O + r0 * D, rows * D, tid, nthr);
      if (o_lt_out) zero_fill(o_lt_out + r0 * D, rows * D, tid, nthr);
      if (o_st_out) zero_fill(o_st_out + r0 * D, rows * D, tid, nthr);
      for (int i = tid; i < rows; i += nthr) {
        if (lse_lt_out) lse_lt_out[r0 + i] = 0.0f;
        if (lse_st_out) lse_st_out[r0 + i] = 0.0f;
      }
    }
    if (n == 0) return;
  }

  // ---- staging, and the largest key norm and value magnitude ----
  float k2 = 0.0f, vm = 0.0f;
  for (int t = T0 + wv; t < NT; t += W) {
    const int r = t * kTile + q;
    float kx[CPL], vx[CPL];
    zero_n(kx);
    zero_n(vx);
    if (r < p.L && r >= p0) {
      load_n<CPL>(K + head_kv + (size_t)r * D + CPL * g, kx);
      load_n<CPL>(V + head_kv + (size_t)r * D + CPL * g, vx);
    }
    store_n<CPL>(Ks + r * LDR + CPL * g, kx);
    store_n<CPL>(Vs + r * LDR + CPL * g, vx);
    k2 = fmaxf(k2, sum_g(dot_n(kx, kx, 0.0f)));
#pragma unroll
    for (int i = 0; i < CPL; ++i) vm = fmaxf(vm, fabsf(vx[i]));
  }
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    k2 = fmaxf(k2, __shfl_xor(k2, off));
    vm = fmaxf(vm, __shfl_xor(vm, off));
  }
  if (lane == 0) {
    red_s[wv] = k2;
    red_s[8 + wv] = vm;
  }
  build_masks<BK, PERPOS, false>(mw, ml, p, sel, bg, p0, tid, nthr);
  __syncthreads();
  k2 = 0.0f;
  vm = 0.0f;
  for (int w = 0; w < W; ++w) {
    k2 = fmaxf(k2, red_s[w]);
    vm = fmaxf(vm, red_s[8 + w]);
  }

  const float c2 = p.scale * kLog2eF;
  const int *kid = reinterpret_cast<const int *>(mw) + ml.kid;
  const int I_lo = max(T0, row_lo / kTile);
  const int n_task = (NT - I_lo) * hpg;

  // query tiles of this wavefront, longest walks first, dealt forth and back over the wavefronts
  for (int rnd = 0; rnd * W < n_task; ++rnd) {
    const int u = rnd * W + ((rnd & 1) ? W - 1 - wv : wv);
    if (u >= n_task) continue;
    const int I = NT - 1 - u / hpg;
    const int bh = bg * hpg + u % hpg;
    const int h = bh % p.H;
    const int iq = I * kTile + q;
    const bool in_range = iq < p.L && iq >= row_lo;
    const bool active = iq < p.L && iq >= p0;
    const size_t rowoff = ((size_t)bh * p.L + min(iq, p.L - 1)) * D;
    const size_t lrow = (size_t)bh * p.L + min(iq, p.L - 1);

    float qf[CPL];
    zero_n(qf);
    if (active) load_n<CPL>(Q + rowoff + CPL * g, qf);
#pragma unroll
    for (int i = 0; i < CPL; ++i) qf[i] *= c2;
    const float q2 = sum_g(dot_n(qf, qf, 0.0f));
    const bool small = __all(q2 * k2 <= kSmallLogit * kSmallLogit) && vm <= 1.0e18f;

    const unsigned long long m_lt = tile_mask(mw, ml.tm_lt, I), m_st = tile_mask(mw, ml.tm_st, I);
    const int kid_q = p.sblk > 0 ? kid[iq] : 0;

    auto logits = [&](int J) -> f32x4 {
      float kf[CPL];
      load_n<CPL>(Ks + (J * kTile + q) * LDR + CPL * g, kf);
      f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < CPL; ++c) s = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c], qf[c], s, 0, 0, 0);
      return s;
    };
    // visibility of this lane's four keys of tile J, one bit each, for the branches that walk the tile
    auto see = [&](int J, bool lt, bool st, unsigned &v_lt, unsigned &v_st) {
      const int key0 = J * kTile + 4 * g;
      unsigned ok = 15u;
      if (J == T0 || J == I || J == NT - 1) {
        ok = 0u;
        const int hi = p.bidir ? p.L - 1 : iq;
#pragma unroll
        for (int r = 0; r < 4; ++r) ok |= (key0 + r >= p0 && key0 + r <= hi) ? 1u << r : 0u;
      }
      v_lt = v_st = 0u;
      if (lt) {
        v_lt = ok;
        if ((PERPOS || BK < kTile) && !dense) {  // the lane's four keys share a block
          const int Jb = key0 / BK;
          const int x = PERPOS ? iq : iq / BK;
          if (((mw[ml.selw + (Jb >> 5) * ml.SR + x] >> (Jb & 31)) & 1u) == 0u) v_lt = 0u;
        }
      }
      if (st) {
        int4 kd = make_int4(0, 0, 0, 0);
        if (p.sblk > 0) kd = *reinterpret_cast<const int4 *>(kid + key0);
        const int kdv[4] = {kd.x, kd.y, kd.z, kd.w};
#pragma unroll
        for (int r = 0; r < 4; ++r) v_st |= st_sees(p, iq - key0 - r, kid_q - kdv[r], key0 + r) ? 1u << r : 0u;
        v_st &= ok;
      }
    };

    float ml_lt = 0.0f, ml_st = 0.0f;  // the references the exponentials are taken against
    if (!small) {
      float a = kNegInfF, c = kNegInfF;
      for (unsigned long long mm = m_lt | m_st; mm; mm &= mm - 1) {
        const int J = __builtin_ctzll(mm);
        const f32x4 s = logits(J);
        unsigned v_lt, v_st;
        see(J, (m_lt >> J) & 1ull, (m_st >> J) & 1ull, v_lt, v_st);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          a = (v_lt >> r) & 1u ? fmaxf(a, s[r]) : a;
          c = (v_st >> r) & 1u ? fmaxf(c, s[r]) : c;
        }
      }
      a = fmaxf(a, __shfl_xor(a, 16));
      a = fmaxf(a, __shfl_xor(a, 32));
      c = fmaxf(c, __shfl_xor(c, 16));
      c = fmaxf(c, __shfl_xor(c, 32));
      ml_lt = a == kNegInfF ? 0.0f : a;
      ml_st = c == kNegInfF ? 0.0f : c;
    }

    f32x4 a_lt[NMB], a_st[NMB];
#pragma unroll
    for (int mb = 0; mb < NMB; ++mb) {
      a_lt[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
      a_st[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    float l_lt = 0.0f, l_st = 0.0f;
    for (unsigned long long mm = m_lt | m_st; mm; mm &= mm - 1) {
      const int J = __builtin_ctzll(mm);
      const bool lt = (m_lt >> J) & 1ull, st = (m_st >> J) & 1ull;
      const f32x4 s = logits(J);
      unsigned v_lt, v_st;
      see(J, lt, st, v_lt, v_st);
      float vf[NMB][4];
#pragma unroll
      for (int mb = 0; mb < NMB; ++mb) col_frag<LDR>(Vs + J * kTile * LDR, g, 16 * mb + q, vf[mb]);
      float e_lt[4], e_st[4];
      if (small) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float e = __builtin_amdgcn_exp2f(s[r]);
          e_lt[r] = (v_lt >> r) & 1u ? e : 0.0f;
          e_st[r] = (v_st >> r) & 1u ? e : 0.0f;
        }
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          e_lt[r] = (v_lt >> r) & 1u ? __builtin_amdgcn_exp2f(s[r] - ml_lt) : 0.0f;
          e_st[r] = (v_st >> r) & 1u ? __builtin_amdgcn_exp2f(s[r] - ml_st) : 0.0f;
        }
      }
      if (lt) {
        l_lt += (e_lt[0] + e_lt[1]) + (e_lt[2] + e_lt[3]);
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int mb = 0; mb < NMB; ++mb)
            a_lt[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[mb][r], e_lt[r], a_lt[mb], 0, 0, 0);
      }
      if (st) {
        l_st += (e_st[0] + e_st[1]) + (e_st[2] + e_st[3]);
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int mb = 0; mb < NMB; ++mb)
            a_st[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[mb][r], e_st[r], a_st[mb], 0, 0, 0);
      }
    }
    // closes a branch: normalised output (zero for rows that take no part), returns the lse
    auto finish = [&](f32x4 (&acc)[NMB], float l, float m) -> float {
      const float lt = sum_g(l);
      const bool ok = active && lt > 0.0f;
      const float inv = ok ? 1.0f / lt : 0.0f;
#pragma unroll
      for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[mb][r] *= inv;
      return ok ? (m + __log2f(lt)) * kLn2F : 0.0f;
    };
    const float lse_lt = finish(a_lt, l_lt, ml_lt);
    if (dense) {
      if (in_range) store_row4<T, D>(O + rowoff, a_lt, g);
      if (in_range && g == 0 && lse_lt_out) lse_lt_out[lrow] = lse_lt;
      continue;
    }
    const float lse_st = finish(a_st, l_st, ml_st);

    // ---- gate and blend (Eq. 18-19) ----
    const float *wl = gate_w + (size_t)h * 2 * D;
    float z = 0.0f;
#pragma unroll
    for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int c = 16 * mb + 4 * g + r;
        if (c < D) {
          z = fmaf(wl[c], a_lt[mb][r], z);
          z = fmaf(wl[D + c], a_st[mb][r], z);
        }
      }
    z = sum_g(z) + (gate_b ? gate_b[h] : 0.0f);
    const float alpha = active ? 1.0f / (1.0f + __expf(-z)) : 0.0f;
    if (in_range) {
      if (o_lt_out) store_row4<float, D>(o_lt_out + rowoff, a_lt, g);
      if (o_st_out) store_row4<float, D>(o_st_out + rowoff, a_st, g);
      f32x4 o[NMB];
#pragma unroll
      for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
        for (int r = 0; r < 4; ++r) o[mb][r] = alpha * a_lt[mb][r] + (1.0f - alpha) * a_st[mb][r];
      store_row4<T, D>(O + rowoff, o, g);
      if (g == 0) {
        if (lse_lt_out) lse_lt_out[lrow] = lse_lt;
        if (lse_st_out) lse_st_out[lrow] = lse_st;
      }
    }
  }
}

// =============================================================================================
// backward: gate pass, dK/dV and dQ of a (row, head), or of the hpg query heads of a (row, group)
// =============================================================================================
// stages: kBwdStage* bits (a subset for callers that run the passes one at a time; the gate pass is redone
// in the workgroup whenever a later pass needs its row constants, and only writes with kBwdStageGate).
// hc: query heads whose Q, dO and row constants are in LDS at a time (hpg whenever that fits).  With hc < hpg
// the key tiles go in rounds of one per wavefront and every round stages the heads chunk by chunk, the
// accumulators staying in registers.
template <typename T, int D, int BK, bool PERPOS>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) void bwd_res_kernel(
    const T *__restrict__ Q, const T *__restrict__ K, const T *__restrict__ V, const int *__restrict__ valid_len,
    const int *__restrict__ sel, const float *__restrict__ gate_w, const float *__restrict__ gate_b,
    const float *__restrict__ o_lt, const float *__restrict__ o_st, const float *__restrict__ lse_lt,
    const float *__restrict__ lse_st, const T *__restrict__ dO, T *__restrict__ dQ, T *__restrict__ dK,
    T *__restrict__ dV, float *__restrict__ partial, int hpg, int hc, unsigned stages, KParams p)
{
  constexpr int CPL = Geo<D>::CPL, NMB = Geo<D>::NMB, LDR = Geo<D>::LDR, GW = 2 * D + 1;
  extern __shared__ __attribute__((aligned(16))) float lds_res[];
  const MaskLayout ml = mask_layout(p, PERPOS, true);
  const int NT = ml.NT, rows = NT * kTile;
  float *A0 = lds_res;                                   // [hc][2][rows][LDR]: Q and dO per head; later K and V
  float *rc = A0 + 2 * hc * rows * LDR + 16;             // [hc][6][rows]: alpha, dz, D_lt, D_st, lse2_lt, lse2_st
  unsigned *mw = reinterpret_cast<unsigned *>(rc + 6 * hc * rows);
  float *red = reinterpret_cast<float *>(mw + ml.words);  // [hc][W][GW]

  const int tid = threadIdx.x, nthr = blockDim.x;
  const int lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), W = nthr >> 6;
  const int bg = blockIdx.x;  // (row, key/value head)
  const int G = p.H / hpg;
  const int b = bg / G;
  const int n = clamp_len(valid_len[b], p.L);
  const int p0 = p.L - n;
  const int T0 = n == 0 ? NT : p0 / kTile;
  const int q = lane & 15, g = lane >> 4;
  const size_t head_kv = (size_t)bg * p.L * D;
  const bool do_gate = stages & kBwdStageGate, do_dq = stages & kBwdStageDQ, do_dkv = stages & kBwdStageDKV;
  const float c2 = p.scale * kLog2eF;

  {  // rows before the first valid tile: zero gradients
    const int zr = min(T0 * kTile, p.L);
    if (do_dkv) {
      zero_fill(dK + head_kv, zr * D, tid, nthr);
      zero_fill(dV + head_kv, zr * D, tid, nthr);
    }
    if (do_dq)
      for (int hh = 0; hh < hpg; ++hh) zero_fill(dQ + (size_t)(bg * hpg + hh) * p.L * D, zr * D, tid, nthr);
    if (n == 0) {
      if (do_gate)
        for (int i = tid; i < hpg * GW; i += nthr) partial[(size_t)bg * hpg * GW + i] = 0.0f;
      return;
    }
  }
  build_masks<BK, PERPOS, true>(mw, ml, p, sel, bg, p0, tid, nthr);
  const int *kid = reinterpret_cast<const int *>(mw) + ml.kid;

  // gate pass of this lane's row of one head: the row constants from its slices of dO, o_lt and o_st
  struct RowConst {
    float al, dz, D_lt, D_st;
  };
  auto row_const = [&](const float (&gr)[CPL], const float (&ol)[CPL], const float (&os)[CPL], const float (&wl)[CPL],
                       const float (&ws)[CPL], float bias, bool valid) -> RowConst {
    const float a_ll = sum_g(dot_n(gr, ol, 0.0f)), a_ss = sum_g(dot_n(gr, os, 0.0f));
    const float w_l = sum_g(dot_n(wl, ol, 0.0f)), w_s = sum_g(dot_n(ws, os, 0.0f));
    RowConst c{0.f, 0.f, 0.f, 0.f};
    if (valid) {
      c.al = 1.0f / (1.0f + __expf(-(bias + w_l + w_s)));
      c.dz = (a_ll - a_ss) * c.al * (1.0f - c.al);
      c.D_lt = c.al * a_ll + c.dz * w_l;
      c.D_st = (1.0f - c.al) * a_ss + c.dz * w_s;
    }
    return c;
  };

  // ---- Q, dO and the row constants of heads h0 .. h0+nh-1 of the group into LDS ----
  auto stage_heads = [&](int h0, int nh, bool gate) {
    for (int hl = 0; hl < nh; ++hl) {
      const int bh = bg * hpg + h0 + hl;
      const int h = bh % p.H;
      float *Qs = A0 + 2 * hl * rows * LDR, *Gs = Qs + rows * LDR, *rch = rc + 6 * hl * rows;
      float wl[CPL], ws[CPL], gl[CPL], gs[CPL], gb = 0.0f;
      load_n<CPL>(gate_w + (size_t)h * 2 * D + CPL * g, wl);
      load_n<CPL>(gate_w + (size_t)h * 2 * D + D + CPL * g, ws);
      const float bias = gate_b ? gate_b[h] : 0.0f;
      zero_n(gl);
      zero_n(gs);
      for (int t = T0 + wv; t < NT; t += W) {
        const int r = t * kTile + q;
        const bool valid = r < p.L && r >= p0;
        const size_t lrow = (size_t)bh * p.L + r, ro = lrow * D + CPL * g;
        float qx[CPL], gr[CPL], ol[CPL], os[CPL];
        zero_n(qx);
        zero_n(gr);
        zero_n(ol);
        zero_n(os);
        float la = kHugeF, lb = kHugeF;  // rows that take no part: every probability zero
        if (valid) {
          load_n<CPL>(Q + ro, qx);
          load_n<CPL>(dO + ro, gr);
          load_n<CPL>(o_lt + ro, ol);
          load_n<CPL>(o_st + ro, os);
          la = lse_lt[lrow] * kLog2eF;
          lb = lse_st[lrow] * kLog2eF;
        }
        store_n<CPL>(Qs + r * LDR + CPL * g, qx);
        store_n<CPL>(Gs + r * LDR + CPL * g, gr);
        const RowConst c = row_const(gr, ol, os, wl, ws, bias, valid);
        if (g == 0) {
          rch[r] = c.al;
          rch[rows + r] = c.dz;
          rch[2 * rows + r] = c.D_lt;
          rch[3 * rows + r] = c.D_st;
          rch[4 * rows + r] = la;
          rch[5 * rows + r] = lb;
        }
        if (gate) {
#pragma unroll
          for (int i = 0; i < CPL; ++i) {
            gl[i] = fmaf(c.dz, ol[i], gl[i]);
            gs[i] = fmaf(c.dz, os[i], gs[i]);
          }
          gb += c.dz;
        }
      }
      if (gate) {  // sums over the 16 rows of the lanes, one slot per wavefront
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) {
#pragma unroll
          for (int i = 0; i < CPL; ++i) {
            gl[i] += __shfl_xor(gl[i], off);
            gs[i] += __shfl_xor(gs[i], off);
          }
          gb += __shfl_xor(gb, off);
        }
        float *rw = red + (hl * W + wv) * GW;
        if (q == 0) {
#pragma unroll
          for (int i = 0; i < CPL; ++i) {
            rw[CPL * g + i] = gl[i];
            rw[D + CPL * g + i] = gs[i];
          }
          if (g == 0) rw[2 * D] = gb;
        }
      }
    }
  };

  // ---- dK, dV: key tiles ----
  if (do_gate || do_dkv) {
    const int chunks = (hpg + hc - 1) / hc;
    int staged = -1;
    for (int rnd = 0; rnd == 0 || (do_dkv && rnd * W < NT - T0); ++rnd) {
      const int u = rnd * W + ((rnd & 1) ? W - 1 - wv : wv);
      const int J = T0 + u;  // early key tiles have the longest walks: they start first
      const bool have = do_dkv && J < NT;
      const int j = min(J, NT - 1) * kTile + q;
      const bool in_range = have && j < p.L;
      const bool key_ok = in_range && j >= p0;
      const int row = min(j, p.L - 1);
      f32x4 dk[NMB], dv[NMB];
#pragma unroll
      for (int mb = 0; mb < NMB; ++mb) {
        dk[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
        dv[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      float kf[CPL], vf[CPL];
      zero_n(kf);
      zero_n(vf);
      if (key_ok) {
        load_n<CPL>(K + head_kv + (size_t)row * D + CPL * g, kf);
        load_n<CPL>(V + head_kv + (size_t)row * D + CPL * g, vf);
      }
#pragma unroll
      for (int i = 0; i < CPL; ++i) kf[i] *= c2;

      for (int ch = 0; ch < chunks; ++ch) {
        const int h0 = ch * hc, nh = min(hc, hpg - h0);
        if (staged != ch) {
          if (staged >= 0) __syncthreads();
          stage_heads(h0, nh, do_gate && rnd == 0);
          staged = ch;
          __syncthreads();  // (covers the masks as well)
          if (do_gate && rnd == 0)
            for (int i = tid; i < nh * GW; i += nthr) {
              const int hl = i / GW, c = i - hl * GW;
              float a = 0.0f;
              for (int w = 0; w < W; ++w) a += red[(hl * W + w) * GW + c];
              partial[(size_t)(bg * hpg + h0 + hl) * GW + c] = a;
            }
        }
        if (!have) continue;
        const unsigned long long m_lt = tile_mask(mw, ml.cm_lt, J), m_st = tile_mask(mw, ml.cm_st, J);
        const int kid_k = p.sblk > 0 ? kid[j] : 0;
        for (int hl = 0; hl < nh; ++hl) {
          const int h = (bg * hpg + h0 + hl) % p.H;
          const float *Qs = A0 + 2 * hl * rows * LDR, *Gs = Qs + rows * LDR, *rch = rc + 6 * hl * rows;
          const float *wrow = gate_w + (size_t)h * 2 * D;
          float wl[CPL], ws[CPL];
          load_n<CPL>(wrow + CPL * g, wl);
          load_n<CPL>(wrow + D + CPL * g, ws);
          const float wv_lt = sum_g(dot_n(wl, vf, 0.0f)), wv_st = sum_g(dot_n(ws, vf, 0.0f));  // Wg_x . v_j
          float t_lt = 0.0f, t_st = 0.0f;  // sum_i dz_i P_ij per branch
          for (unsigned long long mm = m_lt | m_st; mm; mm &= mm - 1) {
            const int I = __builtin_ctzll(mm);
            const bool lt = (m_lt >> I) & 1ull, st = (m_st >> I) & 1ull;
            const int r0 = I * kTile;
            float qa[CPL], ga[CPL];
            load_n<CPL>(Qs + (r0 + q) * LDR + CPL * g, qa);
            load_n<CPL>(Gs + (r0 + q) * LDR + CPL * g, ga);
            f32x4 s = {0.f, 0.f, 0.f, 0.f}, gv = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
              s = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[c], kf[c], s, 0, 0, 0);
              gv = __builtin_amdgcn_mfma_f32_16x16x4f32(ga[c], vf[c], gv, 0, 0, 0);
            }
            const int i0 = r0 + 4 * g;  // this lane's rows i0 .. i0+3
            unsigned ok = 15u;
            if (I == J && !p.bidir) {
              ok = 0u;
#pragma unroll
              for (int r = 0; r < 4; ++r) ok |= i0 + r >= j ? 1u << r : 0u;
            }
            float al[4], dz[4], pc[4], ds[4];
            load_n<4>(rch + i0, al);
            load_n<4>(rch + rows + i0, dz);
            zero_n(pc);
            zero_n(ds);
            if (lt) {
              float Dx[4], l2[4];
              load_n<4>(rch + 2 * rows + i0, Dx);
              load_n<4>(rch + 4 * rows + i0, l2);
              unsigned v = ok;
              const int Jb = j / BK;
              if (PERPOS) {
                const uint4 w4 = *reinterpret_cast<const uint4 *>(mw + ml.selw + (Jb >> 5) * ml.SR + i0);
                const unsigned wr[4] = {w4.x, w4.y, w4.z, w4.w};
                unsigned sb = 0u;
#pragma unroll
                for (int r = 0; r < 4; ++r) sb |= ((wr[r] >> (Jb & 31)) & 1u) << r;
                v &= sb;
              } else if (BK < kTile) {
                if (((mw[ml.selw + (Jb >> 5) * ml.SR + i0 / BK] >> (Jb & 31)) & 1u) == 0u) v = 0u;
              }
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const float pr = (v >> r) & 1u ? __builtin_amdgcn_exp2f(s[r] - l2[r]) : 0.0f;
                pc[r] = al[r] * pr;
                ds[r] = pr * fmaf(al[r], gv[r], fmaf(dz[r], wv_lt, -Dx[r]));
                t_lt = fmaf(dz[r], pr, t_lt);
              }
            }
            if (st) {
              float Dx[4], l2[4];
              load_n<4>(rch + 3 * rows + i0, Dx);
              load_n<4>(rch + 5 * rows + i0, l2);
              int4 kd = make_int4(0, 0, 0, 0);
              if (p.sblk > 0) kd = *reinterpret_cast<const int4 *>(kid + i0);
              const int kdv[4] = {kd.x, kd.y, kd.z, kd.w};
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const bool v = ((ok >> r) & 1u) && st_sees(p, i0 + r - j, kdv[r] - kid_k, j);
                const float pr = v ? __builtin_amdgcn_exp2f(s[r] - l2[r]) : 0.0f;
                const float as = 1.0f - al[r];
                pc[r] = fmaf(as, pr, pc[r]);
                ds[r] = fmaf(pr, fmaf(as, gv[r], fmaf(dz[r], wv_st, -Dx[r])), ds[r]);
                t_st = fmaf(dz[r], pr, t_st);
              }
            }
            // dV^T += dO^T (a P), dK^T += Q^T dS: row = query 4g + r, column = channel 16*mb + q
            float gc[NMB][4], qc[NMB][4];
#pragma unroll
            for (int mb = 0; mb < NMB; ++mb) {
              col_frag<LDR>(Gs + r0 * LDR, g, 16 * mb + q, gc[mb]);
              col_frag<LDR>(Qs + r0 * LDR, g, 16 * mb + q, qc[mb]);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
              for (int mb = 0; mb < NMB; ++mb) {
                dv[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(gc[mb][r], pc[r], dv[mb], 0, 0, 0);
                dk[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(qc[mb][r], ds[r], dk[mb], 0, 0, 0);
              }
          }
          // the gate part of dV: sum_i dz_i P_ij times the gate row of the branch
          t_lt = sum_g(t_lt);
          t_st = sum_g(t_st);
#pragma unroll
          for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int c = 16 * mb + 4 * g + r;
              if (c < D) dv[mb][r] += fmaf(t_lt, wrow[c], t_st * wrow[D + c]);
            }
        }
      }
      if (in_range) {
        store_grad_row<T, D>(dK + head_kv + (size_t)row * D, dk, p.scale, key_ok, p, true, row, g);
        store_grad_row<T, D>(dV + head_kv + (size_t)row * D, dv, 1.0f, key_ok, p, false, row, g);
      }
    }
  }

  // ---- dQ: query tiles ----
  if (!do_dq) return;
  const bool have_rc = (do_gate || do_dkv) && hc >= hpg;  // the row constants of every head are in LDS
  float *Ks = A0, *Vs = A0 + rows * LDR;
  __syncthreads();
  for (int t = T0 + wv; t < NT; t += W) {
    const int r = t * kTile + q;
    float kx[CPL], vx[CPL];
    zero_n(kx);
    zero_n(vx);
    if (r < p.L && r >= p0) {
      load_n<CPL>(K + head_kv + (size_t)r * D + CPL * g, kx);
      load_n<CPL>(V + head_kv + (size_t)r * D + CPL * g, vx);
    }
    store_n<CPL>(Ks + r * LDR + CPL * g, kx);
    store_n<CPL>(Vs + r * LDR + CPL * g, vx);
  }
  __syncthreads();
  const int n_task = (NT - T0) * hpg;
  for (int rnd = 0; rnd * W < n_task; ++rnd) {
    const int u = rnd * W + ((rnd & 1) ? W - 1 - wv : wv);
    if (u >= n_task) continue;
    const int I = NT - 1 - u / hpg;
    const int hh = u % hpg;
    const int bh = bg * hpg + hh;
    const int h = bh % p.H;
    const int iq = I * kTile + q;
    const bool in_range = iq < p.L;
    const bool active = in_range && iq >= p0;
    const int row = min(iq, p.L - 1);
    const size_t lrow = (size_t)bh * p.L + row, rowoff = lrow * D;
    float qf[CPL], gr[CPL], wl[CPL], ws[CPL];
    zero_n(qf);
    zero_n(gr);
    load_n<CPL>(gate_w + (size_t)h * 2 * D + CPL * g, wl);
    load_n<CPL>(gate_w + (size_t)h * 2 * D + D + CPL * g, ws);
    if (active) {
      load_n<CPL>(Q + rowoff + CPL * g, qf);
      load_n<CPL>(dO + rowoff + CPL * g, gr);
    }
#pragma unroll
    for (int i = 0; i < CPL; ++i) qf[i] *= c2;
    RowConst c;
    float l2_lt, l2_st;
    if (have_rc) {
      const float *rch = rc + 6 * hh * rows;
      c.al = rch[iq];
      c.dz = rch[rows + iq];
      c.D_lt = rch[2 * rows + iq];
      c.D_st = rch[3 * rows + iq];
      l2_lt = rch[4 * rows + iq];
      l2_st = rch[5 * rows + iq];
    } else {
      float ol[CPL], os[CPL];
      zero_n(ol);
      zero_n(os);
      if (active) {
        load_n<CPL>(o_lt + rowoff + CPL * g, ol);
        load_n<CPL>(o_st + rowoff + CPL * g, os);
      }
      c = row_const(gr, ol, os, wl, ws, gate_b ? gate_b[h] : 0.0f, active);
      l2_lt = active ? lse_lt[lrow] * kLog2eF : kHugeF;
      l2_st = active ? lse_st[lrow] * kLog2eF : kHugeF;
    }
    float gx_lt[CPL], gx_st[CPL];  // dO_x of this lane's row
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
      gx_lt[i] = fmaf(c.al, gr[i], c.dz * wl[i]);
      gx_st[i] = fmaf(1.0f - c.al, gr[i], c.dz * ws[i]);
    }
    f32x4 dq[NMB];
#pragma unroll
    for (int mb = 0; mb < NMB; ++mb) dq[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
    const unsigned long long m_lt = tile_mask(mw, ml.tm_lt, I), m_st = tile_mask(mw, ml.tm_st, I);
    const int kid_q = p.sblk > 0 ? kid[iq] : 0;
    for (unsigned long long mm = m_lt | m_st; mm; mm &= mm - 1) {
      const int J = __builtin_ctzll(mm);
      const bool lt = (m_lt >> J) & 1ull, st = (m_st >> J) & 1ull;
      float kf[CPL], vf[CPL];
      load_n<CPL>(Ks + (J * kTile + q) * LDR + CPL * g, kf);
      load_n<CPL>(Vs + (J * kTile + q) * LDR + CPL * g, vf);
      f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < CPL; ++i) s = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[i], qf[i], s, 0, 0, 0);
      const int key0 = J * kTile + 4 * g;
      unsigned ok = 15u;
      if (J == T0 || J == I || J == NT - 1) {
        ok = 0u;
        const int hi = p.bidir ? p.L - 1 : iq;
#pragma unroll
        for (int r = 0; r < 4; ++r) ok |= (key0 + r >= p0 && key0 + r <= hi) ? 1u << r : 0u;
      }
      float ds[4];
      zero_n(ds);
      if (lt) {
        f32x4 gv = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < CPL; ++i) gv = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[i], gx_lt[i], gv, 0, 0, 0);
        unsigned v = ok;
        if (PERPOS || BK < kTile) {
          const int Jb = key0 / BK;
          const int x = PERPOS ? iq : iq / BK;
          if (((mw[ml.selw + (Jb >> 5) * ml.SR + x] >> (Jb & 31)) & 1u) == 0u) v = 0u;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
          ds[r] = (v >> r) & 1u ? __builtin_amdgcn_exp2f(s[r] - l2_lt) * (gv[r] - c.D_lt) : 0.0f;
      }
      if (st) {
        f32x4 gv = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < CPL; ++i) gv = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[i], gx_st[i], gv, 0, 0, 0);
        int4 kd = make_int4(0, 0, 0, 0);
        if (p.sblk > 0) kd = *reinterpret_cast<const int4 *>(kid + key0);
        const int kdv[4] = {kd.x, kd.y, kd.z, kd.w};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const bool v = ((ok >> r) & 1u) && st_sees(p, iq - key0 - r, kid_q - kdv[r], key0 + r);
          const float e = v ? __builtin_amdgcn_exp2f(s[r] - l2_st) : 0.0f;
          ds[r] = fmaf(e, gv[r] - c.D_st, ds[r]);
        }
      }
      float kc[NMB][4];
#pragma unroll
      for (int mb = 0; mb < NMB; ++mb) col_frag<LDR>(Ks + J * kTile * LDR, g, 16 * mb + q, kc[mb]);
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int mb = 0; mb < NMB; ++mb)
          dq[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(kc[mb][r], ds[r], dq[mb], 0, 0, 0);
    }
    if (in_range) store_grad_row<T, D>(dQ + rowoff, dq, p.scale, active, p, true, row, g);
  }
}

// =============================================================================================
// launchers
// =============================================================================================
namespace {

int res_rows(const KParams &p) { return (p.L + kTile - 1) / kTile * kTile; }
size_t res_fwd_lds_bytes(const KParams &p, bool perpos)
{
  return ((size_t)2 * res_rows(p) * (p.d + 4) + 16 + mask_layout(p, perpos, false).words) * sizeof(float);
}
size_t res_bwd_lds_bytes(const KParams &p, bool perpos, int hc, int waves)
{
  return ((size_t)2 * hc * res_rows(p) * (p.d + 4) + 16 + (size_t)6 * hc * res_rows(p) + mask_layout(p, perpos, true).words +
          (size_t)hc * waves * (2 * p.d + 1)) * sizeof(float);
}

bool res_shape(const KParams &p)
{
  // One workgroup per (row, head): enough of them to fill the chip, or so little work that it does not matter.
  return (p.d == 8 || p.d == 16 || p.d == 32) && (p.b == 8 || p.b == 16) && p.L <= kMaxTiles * kTile &&
         ((long)p.B * p.H >= 64 || p.L <= 256);
}

constexpr int kResWaves = 8;
// The per-position form has limits that its callers know (144 KB of fp32 rows of 20 or 36 floats, see the header).
constexpr size_t kPosLdsLimit = 144 * 1024;
size_t pos_fwd_limit_bytes(const KParams &p) { return 2 * (size_t)(p.NB * p.b + 16) * ((p.d < 16 ? 16 : p.d) + 4) * sizeof(float); }
size_t pos_bwd_limit_bytes(const KParams &p)
{
  const size_t rows = (size_t)(p.NB * p.b + 16);
  return pos_fwd_limit_bytes(p) + 6 * rows * sizeof(float) + (rows + p.NB) * sizeof(unsigned long long);
}

// (more than 64 KB of dynamic LDS has to be asked for; where it is not granted the launch fails and the
// entry point reports it)
template <typename Kern>
void want_lds(Kern kernel, size_t lds)
{
  if (lds > 64 * 1024)
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

template <typename F>
void with_res_dims(const KParams &p, F &&f)
{
  auto with_bk = [&](auto dim) {
    if (p.b == 8) f(dim, std::integral_constant<int, 8>{});
    else f(dim, std::integral_constant<int, 16>{});
  };
  if (p.d == 8) with_bk(std::integral_constant<int, 8>{});
  else if (p.d == 16) with_bk(std::integral_constant<int, 16>{});
  else with_bk(std::integral_constant<int, 32>{});
}

}  // namespace

bool fwd_res_supported(const KParams &p, int dtype)
{
  (void)dtype;
  return res_shape(p) && res_fwd_lds_bytes(p, false) <= kResLdsMax - 256;
}

// the per-position form exists in this kernel family only: what the shape has to satisfy, whatever the batch
bool fwd_positions_supported(const KParams &p, int dtype)
{
  (void)dtype;
  return (p.d == 8 || p.d == 16 || p.d == 32) && (p.b == 8 || p.b == 16) && !p.bidir && p.NB <= 64 && p.nq == p.NB &&
         pos_fwd_limit_bytes(p) <= kPosLdsLimit;
}

bool bwd_res_supported(const KParams &p, int dtype)
{
  (void)dtype;
  return res_shape(p) && res_bwd_lds_bytes(p, false, 1, kResWaves) <= kResLdsMax - 256;
}

bool bwd_positions_supported(const KParams &p, int dtype)
{
  return fwd_positions_supported(p, dtype) && pos_bwd_limit_bytes(p) <= kPosLdsLimit;
}

template <typename T>
static void launch_fwd_res_t(const KParams &p, const FwdArgs &a, hipStream_t st)
{
  const bool perpos = a.kv_groups > 0;
  const size_t lds = res_fwd_lds_bytes(p, perpos);
  const int hpg = perpos ? p.H / a.kv_groups : 1;
  with_res_dims(p, [&](auto dim, auto bk) {
    constexpr int D = decltype(dim)::value, BK = decltype(bk)::value;
    auto go = [&](auto kernel) {
      want_lds(kernel, lds);
      hipLaunchKernelGGL(kernel, dim3((unsigned)(p.B * p.H / hpg)), dim3(64 * kResWaves), lds, st, (const T *)a.Q,
                         (const T *)a.K, (const T *)a.V, a.valid_len, a.dense ? nullptr : a.sel, a.gate_w, a.gate_b, (T *)a.O,
                         (float *)a.o_lt, (float *)a.o_st, a.lse_lt, a.lse_st, hpg, p);
    };
    if (perpos) go(fwd_res_kernel<T, D, BK, true>);
    else go(fwd_res_kernel<T, D, BK, false>);
  });
}

void launch_fwd_res(const KParams &p, int dtype, const FwdArgs &a, hipStream_t st)
{
  if (dtype == 0) launch_fwd_res_t<float>(p, a, st);
  else launch_fwd_res_t<bf16_t>(p, a, st);
}

template <typename T>
static void launch_bwd_res_t(const KParams &p, const BwdArgs &a, const BwdWorkspace &w, unsigned stages, int kv_groups,
                             hipStream_t st)
{
  const bool perpos = kv_groups > 0;
  const int hpg = perpos ? p.H / kv_groups : 1;
  int hc = hpg;  // as many heads of the group at a time as fit
  while (hc > 1 && res_bwd_lds_bytes(p, perpos, hc, kResWaves) > kResLdsMax - 256) --hc;
  const size_t lds = res_bwd_lds_bytes(p, perpos, hc, kResWaves);
  with_res_dims(p, [&](auto dim, auto bk) {
    constexpr int D = decltype(dim)::value, BK = decltype(bk)::value;
    auto go = [&](auto kernel) {
      want_lds(kernel, lds);
      hipLaunchKernelGGL(kernel, dim3((unsigned)(p.B * p.H / hpg)), dim3(64 * kResWaves), lds, st, (const T *)a.Q,
                         (const T *)a.K, (const T *)a.V, a.valid_len, a.sel, a.gate_w, a.gate_b, (const float *)a.o_lt,
                         (const float *)a.o_st, a.lse_lt, a.lse_st, (const T *)a.dO, (T *)a.dQ, (T *)a.dK, (T *)a.dV,
                         w.partial, hpg, hc, stages, p);
    };
    if (perpos) go(bwd_res_kernel<T, D, BK, true>);
    else go(bwd_res_kernel<T, D, BK, false>);
  });
}

// gate pass (partial gate gradients, one row of 2d+1 per (row, head), in w.partial), dK/dV and dQ as asked for;
// kv_groups > 0: a.sel holds one row per position and group
void launch_bwd_res(const KParams &p, int dtype, const BwdArgs &a, const BwdWorkspace &w, unsigned stages, int kv_groups,
                    hipStream_t st)
{
  if ((stages & (kBwdStageGate | kBwdStageDQ | kBwdStageDKV)) == 0) return;
  if (dtype == 0) launch_bwd_res_t<float>(p, a, w, stages, kv_groups, st);
  else launch_bwd_res_t<bf16_t>(p, a, w, stages, kv_groups, st);
}

}  // namespace blossom
