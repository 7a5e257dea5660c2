// Forward and backward on the fp32 matrix instructions for small heads (Eq. 1 under the two branch masks,
// Eq. 16-19 and their chain rule, and the same-style dense causal comparison): fp32 or bf16 storage,
// d in {8, 16, 32}, block size 8 or 16.  That is the paper's own regime (Sec. 4.1, Appendix E: hidden size 64
// or 128 over 2 to 8 heads, selection block 16, histories of 200 items, up to 2000 in the efficiency study);
// the 64 x 64 bf16 tiles of the other matrix-core kernels would be mostly padding there.
//
// Positions are cut into 16-row tiles of v_mfma_f32_16x16x4_f32 (true fp32 products accumulated in fp32; d = 8: contractions over
// rows as 4x4 blocks; bf16 storage from d = 16 on: the bf16 matrix instructions with the same accuracy; see THE MATRIX OPERANDS)
// whatever the block size; a selection block of 8 is half a tile and the selection is tested per element.
// A wavefront takes one query tile (forward, dQ) or one key tile (dK/dV) at a time.  Heads that fit a workgroup's LDS
// (small_lds_limit; fp32: L up to 256 at d = 32, 272 at d = 16, 688 at d = 8, less in the backward) are staged
// there, and the backward of such a head is one kernel that reads every tensor once; longer ones stream the tiles
// they walk from memory (L1 and L2) into operand registers, with neither barriers nor a limit on the length.
//
// BOTH BRANCHES IN ONE WALK.  The branches share the logits, so a walk visits the union of the two tile
// sets once and applies two masks to one product: forward forms S once and adds P_lt V and P_st V;
// backward needs one product each for dQ, dK and dV, because dS = dS_lt + dS_st multiplies the same K and Q (dV:
// the coefficient of dO is a_lt P_lt + a_st P_st, the gate part is a rank-one term per key).  The tiles of a walk
// come from bit words over tiles: the short-term ones by a ballot of the mask geometry, the long-term ones
// from the selection rows.
//   forward: S^T = K Q^T, keys as the M dimension: lane (q = lane % 16, g = lane / 16) owns query column
//            q and the logits of keys 4g .. 4g+3 of the tile; O^T += V^T P^T with P^T = the accumulator of
//            S^T as it stands (step r contracts key 4g + r of every lane group).
//   dQ:      same orientation: S^T and G_x^T = V dO_x^T leave the matrix cores in the layout in which
//            dS^T is the B operand of dQ^T += K^T dS^T.
//   dK/dV:   queries as the M dimension (lane (key, g): key column, query rows 4g .. 4g+3).
// A contraction over channels takes channel (d/4)*g + s in step s, so that a lane's operands are d/4
// consecutive elements: one or two 16-byte loads per tile.
//
// EXPONENTIALS WITHOUT A RUNNING MAXIMUM.  A walk takes exp2 of the logits themselves, one exponential for both
// branches, and keeps the largest |logit| it met (of masked keys too): up to 60 (log2 units) nothing overflows or loses
// accuracy in fp32.  Beyond that (or if an output left fp32's range) the walk is repeated with the two row maxima,
// found by a walk of their own, as references.  With every tile beyond it the forward of the near form (see there) takes 29 us instead of 16
// at B=256 H=2 L=200 d=32, 493 instead of 185 at B=2048 H=8 L=200 d=16, 184 instead of 43 at B=32 H=8 L=2000 d=8; the general one there 30
// and 17, 529 and 243, 191 and 51.
//
// VALUES THAT ARE NOT FINITE.  A walk multiplies whole tiles, so a masked element adds zero times whatever the tile holds: a NaN
// or an infinity, in a row of the padding too, would reach every row of its tile.  Such a result is not finite itself,
// which a few instructions at the end of a walk tell; the walk is then repeated with those elements taken out of the
// products, and the rows that do see one of them get NaN.  (dQ of a head in LDS: taken out as the head is staged.)
//
// The dQ kernel also does the per-row gate pass (alpha, dz, D_x and the gate-weight gradients): a wavefront has
// its query rows' dO at hand.  It leaves the row constants and the long-term tile words of every query tile for the
// dK/dV kernel, which finds the query tiles of a key tile by a ballot over those words (no inverse lists).
// With dO_x = a_x*dO + dz*Wg_x the upstream gradient of branch x (a_lt = alpha, a_st = 1 - alpha) and D_x = dO_x.o_x:
//   P_ij = exp(scale*q_i.k_j - lse_x,i),  dS_ij = P_ij * (dO_x,i.v_j - D_x,i),
//   dQ_i = scale * sum_j dS_ij k_j,  dK_j = scale * sum_i dS_ij q_i,  dV_j = sum_i P_ij dO_x,i.
// Masks (the causal window, or all of Eq. 15 in its causal or its bidirectional form), gate, outputs and padding
// rules are those of the scalar kernels of generic.hip; shapes outside this range stay there.
#include <algorithm>

#include "launch.h"
#include "mfma_common.h"
#include "near_host.h"

namespace blossom {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr float kLog2eF = 1.4426950408889634f;
constexpr float kLn2F = 0.6931471805599453f, kLn2Low = (float)(0.6931471805599453 - (double)kLn2F);  // ln 2 in two parts
constexpr float kNegInfF = -__builtin_huge_valf();
constexpr float kHugeF = 1.0e30f;
constexpr int kTile = 16;
constexpr int kMaxWaves = 8;          // wavefronts per workgroup at most
constexpr float kSmallLogit = 60.0f;  // log2 units: exp2 of such a logit, and sums over a row, stay far inside fp32

template <int D>
struct Geo {
  static constexpr int CPL = D / 4;            // channels per lane of a channel contraction: CPL*g .. CPL*g + CPL-1
  static constexpr int NMB = (D + 15) / 16;    // 16-channel output blocks (d = 8 fills half of one)
  static constexpr bool kQuads = D == 8;       // contractions over rows by quads of channels (Operands::add)
  static constexpr int NACC = kQuads ? 2 : NMB;  // their accumulators
};

// both halves, the lower one first; at: 8-byte aligned
__device__ __forceinline__ void store_pair(unsigned *at, unsigned long long x)
{
  *reinterpret_cast<uint2 *>(at) = make_uint2((unsigned)x, (unsigned)(x >> 32));
}
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
// Waits for what these registers are loaded with.  (Each goes to the assembly in its own type: through a pointer to another one the
// compiler need not see that they are read and written here.)
template <typename X, int N>
__device__ __forceinline__ void arrive(X (&x)[N])
{
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+v"(x[i]));
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
// reciprocal to fp32 accuracy: the hardware estimate (1 ulp) and one Newton step; x is a normal number
__device__ __forceinline__ float recip(float x)
{
  const float r = __builtin_amdgcn_rcpf(x);
  return fmaf(r, fmaf(-x, r, 1.0f), r);
}
// (a comparison and not fminf, which would turn a NaN into 126 and the gate into a finite number)
__device__ __forceinline__ float sigmoid(float z)
{
  const float x = -z * kLog2eF;
  return recip(1.0f + __builtin_amdgcn_exp2f(x > 126.0f ? 126.0f : x));
}

// sum and maximum over the four lane groups of a column (rows 0/1, 2/3 then halves of the wavefront swapped in
// registers), sum over the 16 columns of a lane group (rotations inside a row of 16 lanes)
typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));
template <typename F>
__device__ __forceinline__ float fold_g(float x, F &&f)
{
  const unsigned u = __float_as_uint(x);
  const u32x2_t a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const unsigned v = __float_as_uint(f(__uint_as_float(a[0]), __uint_as_float(a[1])));
  const u32x2_t b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return f(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float sum_g(float x)
{
  return fold_g(x, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ float max_g(float x)
{
  return fold_g(x, [](float a, float b) { return fmaxf(a, b); });
}
template <int N>
__device__ __forceinline__ float row_ror(float x)
{
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 + N, 0xf, 0xf, false));
}
__device__ __forceinline__ float sum_row(float x)
{
  x += row_ror<8>(x);
  x += row_ror<4>(x);
  x += row_ror<2>(x);
  return x + row_ror<1>(x);
}
__device__ __forceinline__ bool finite(float x) { return fabsf(x) <= 3.402823466e38f; }

// THE MATRIX OPERANDS.  Row: a lane's channels of one row, for contractions over channels; Col: its four rows of one channel, for
// contractions over rows, whose other side is four fp32 coefficients; Split: a row of fp32 values.
// fp32 storage, and bf16 at d = 8: floats for v_mfma_f32_16x16x4_f32.
// bf16 storage from d = 16 on: the stored bits for v_mfma_f32_16x16x16_bf16 and 16x16x32, one instruction where the fp32 form takes four
// or eight, at half the cycles: products of two stored rows are exact either way, and an fp32 side enters as the exact sum of three
// bf16 terms.  (Against 64 bits the bf16 forms err less, sums of 32 products 2.9e-8 against 3.5e-8, three-term ones of 16
// 3.3e-8 against 7.3e-8: they round once per instruction.)  At d = 16 a contraction over rows would save nothing: the split
// of its coefficients takes 22 vector instructions.  A training step at B=256 H=2 L=200 d=32 in the bidirectional form: 145 us
// with everything as floats, 89 like this.
constexpr bool stored_bits(bool bf16, int d) { return bf16 && d >= 16; }
template <typename T, int D>
struct Operands {
  static constexpr bool kBf = stored_bits(std::is_same<T, bf16_t>::value, D), kBfCol = kBf && D == 32;
  static constexpr int CPL = Geo<D>::CPL;
  struct RowF { float v[CPL]; };
  struct RowB { unsigned w[CPL / 2]; };
  struct ColF { float v[4]; };
  struct ColB { unsigned w[2]; };
  using Row = std::conditional_t<kBf, RowB, RowF>;
  using Col = std::conditional_t<kBfCol, ColB, ColF>;
  struct Split { Row term[kBf ? 3 : 1]; };

  static __device__ __forceinline__ void floats(const Row &a, float (&o)[CPL])
  {
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
      if constexpr (kBf) o[i] = __uint_as_float((i & 1) ? a.w[i / 2] & 0xFFFF0000u : a.w[i / 2] << 16);
      else o[i] = a.v[i];
    }
  }
  static __device__ __forceinline__ void arrived(Row &a)
  {
    if constexpr (kBf) arrive(a.w);
    else arrive(a.v);
  }
  static __device__ __forceinline__ void clean(Row &a)  // elements that are not finite become zeros
  {
    if constexpr (kBf) {
#pragma unroll
      for (int i = 0; i < CPL / 2; ++i) {
        a.w[i] &= (a.w[i] & 0x7F80u) == 0x7F80u ? 0xFFFF0000u : ~0u;
        a.w[i] &= (a.w[i] & 0x7F800000u) == 0x7F800000u ? 0xFFFFu : ~0u;
      }
    } else {
#pragma unroll
      for (int i = 0; i < CPL; ++i) a.v[i] = finite(a.v[i]) ? a.v[i] : 0.0f;
    }
  }
  // what the query (or key) side of the logits is multiplied by before (kBf: the logits themselves, after)
  static __device__ __forceinline__ void scale(Row &a, float c)
  {
    if constexpr (!kBf) {
#pragma unroll
      for (int i = 0; i < CPL; ++i) a.v[i] *= c;
    }
  }
  static __device__ __forceinline__ f32x4 dot(const Row &a, const Row &b, f32x4 c)
  {
    if constexpr (kBf && D == 32) {
      return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(mfma::bf16x8, a), __builtin_bit_cast(mfma::bf16x8, b), c, 0, 0, 0);
    } else if constexpr (kBf) {
      return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(mfma::s16x4, a), __builtin_bit_cast(mfma::s16x4, b), c, 0, 0, 0);
    } else {
#pragma unroll
      for (int i = 0; i < CPL; ++i) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[i], b.v[i], c, 0, 0, 0);
      return c;
    }
  }
  static __device__ __forceinline__ f32x4 dot(const Row &a, const Split &b, f32x4 c)
  {
    if constexpr (kBf) c = dot(a, b.term[1], dot(a, b.term[2], c));
    return dot(a, b.term[0], c);
  }
  // x, y -> their upper halves in one register, what is left of them
  static __device__ __forceinline__ unsigned upper(float &x, float &y)
  {
    const unsigned a = __float_as_uint(x), b = __float_as_uint(y);
    x -= __uint_as_float(a & 0xFFFF0000u);
    y -= __uint_as_float(b & 0xFFFF0000u);
    return __builtin_amdgcn_perm(b, a, 0x07060302u);
  }
  static __device__ __forceinline__ Split split(const float (&x)[CPL])
  {
    Split s;
    if constexpr (kBf) {
#pragma unroll
      for (int i = 0; i < CPL; i += 2) {
        float a = x[i], b = x[i + 1];
#pragma unroll
        for (int t = 0; t < 3; ++t) s.term[t].w[i / 2] = upper(a, b);
      }
    } else {
#pragma unroll
      for (int i = 0; i < CPL; ++i) s.term[0].v[i] = x[i];
    }
    return s;
  }
  // acc += sum over the lanes' rows of e times the operand
  // d = 8: sixteen blocks of 4x4 in one instruction, the operand's quad of channels 4h .. 4h+3 handed to the four blocks of a lane
  // group.  Lane (q, g) then holds the part of the sum over its rows 4g .. 4g+3 (channel 4h + r of row q in acc[h][r]; total()
  // closes it): half the matrix cores' time of the 16-row form, of which d = 8 fills half, and sums that err less (dK at L=1000:
  // 2.8e-7 against 3.3e-7).  With the distances taken by lane groups (add_row), B=32 H=8 L=2000: dK/dV 129 -> 103 us, dQ 79 -> 69.
  static __device__ __forceinline__ void add(const Col (&a)[Geo<D>::NMB], const float (&e)[4], f32x4 (&acc)[Geo<D>::NACC])
  {
    if constexpr (Geo<D>::kQuads) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        acc[0] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[0].v[r], e[r], acc[0], 2, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[0].v[r], e[r], acc[1], 2, 1, 0);
      }
    } else if constexpr (kBfCol) {
      ColB c[3];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        float x = e[2 * i], y = e[2 * i + 1];
#pragma unroll
        for (int t = 0; t < 3; ++t) c[t].w[i] = upper(x, y);
      }
#pragma unroll
      for (int t = 2; t >= 0; --t)
#pragma unroll
        for (int mb = 0; mb < Geo<D>::NMB; ++mb)
          acc[mb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(mfma::s16x4, a[mb]), __builtin_bit_cast(mfma::s16x4, c[t]),
                                                              acc[mb], 0, 0, 0);
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int mb = 0; mb < Geo<D>::NMB; ++mb) acc[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[mb].v[r], e[r], acc[mb], 0, 0, 0);
    }
  }
  static __device__ __forceinline__ Col col(float x0, float x1, float x2, float x3)  // (of stored values)
  {
    if constexpr (kBfCol) return ColB{{upper(x0, x1), upper(x2, x3)}};
    else return ColF{{x0, x1, x2, x3}};
  }
};

constexpr float kNaN = __builtin_nanf("");
// Takes the elements that are not finite out of a tile's operand (element r of lane (q, g): row 4g + r).  lost[r]: NaN where that
// row held one, to be added to its coefficient in the columns that see the row, else 0.
template <typename T, int D>
__device__ __forceinline__ void take_out(typename Operands<T, D>::Col (&a)[Geo<D>::NMB], int g, float (&lost)[4])
{
  float x[Geo<D>::NMB][4];
  bool here[4] = {false, false, false, false};
#pragma unroll
  for (int mb = 0; mb < Geo<D>::NMB; ++mb) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if constexpr (Operands<T, D>::kBfCol) x[mb][r] = __uint_as_float((r & 1) ? a[mb].w[r / 2] & 0xFFFF0000u : a[mb].w[r / 2] << 16);
      else x[mb][r] = a[mb].v[r];
      here[r] |= !finite(x[mb][r]);
      x[mb][r] = finite(x[mb][r]) ? x[mb][r] : 0.0f;
    }
    a[mb] = Operands<T, D>::col(x[mb][0], x[mb][1], x[mb][2], x[mb][3]);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) lost[r] = ((__ballot(here[r]) >> (16 * g)) & 0xFFFFull) != 0ull ? kNaN : 0.0f;
}
template <int N>
__device__ __forceinline__ float abs_sum(const f32x4 (&a)[N])
{
  float x = 0.0f;
#pragma unroll
  for (int mb = 0; mb < N; ++mb)
#pragma unroll
    for (int r = 0; r < 4; ++r) x += fabsf(a[mb][r]);
  return x;
}
template <int N>
__device__ __forceinline__ void clear(f32x4 (&a)[N])
{
#pragma unroll
  for (int mb = 0; mb < N; ++mb) a[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
}

// the sums over all lane groups, as the accumulators of the 16-row form hold them: channel 16*mb + 4g + r (modulo 8 at d = 8)
template <int D>
__device__ __forceinline__ void total(const f32x4 (&a)[Geo<D>::NACC], f32x4 (&o)[Geo<D>::NMB])
{
  if constexpr (Geo<D>::kQuads) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const u32x2_t x = __builtin_amdgcn_permlane16_swap(__float_as_uint(a[0][r]), __float_as_uint(a[1][r]), false, false);
      const unsigned y = __float_as_uint(__uint_as_float(x[0]) + __uint_as_float(x[1]));
      const u32x2_t z = __builtin_amdgcn_permlane32_swap(y, y, false, false);
      o[0][r] = __uint_as_float(z[0]) + __uint_as_float(z[1]);
    }
  } else {
#pragma unroll
    for (int mb = 0; mb < Geo<D>::NMB; ++mb) o[mb] = a[mb];
  }
}

// four elements that the caches need not keep
__device__ __forceinline__ void store4_once(float *p, const float (&o)[4])
{
  const f32x4 v = {o[0], o[1], o[2], o[3]};
  __builtin_nontemporal_store(v, reinterpret_cast<f32x4 *>(p));
}
__device__ __forceinline__ void store4_once(bf16_t *p, const float (&o)[4])
{
  typedef unsigned u32x2_once __attribute__((ext_vector_type(2)));
  const u32x2_once v = {(uint32_t)f32_to_bf16(o[0]) | ((uint32_t)f32_to_bf16(o[1]) << 16),
                        (uint32_t)f32_to_bf16(o[2]) | ((uint32_t)f32_to_bf16(o[3]) << 16)};
  __builtin_nontemporal_store(v, reinterpret_cast<u32x2_once *>(p));
}

// lane (col, g) holds channels 16*mb + 4g + r of one row in a[mb][r]: stores those below D
// ONCE: a branch output, read by one later kernel if at all.  Those and the gradients written past the caches leave them to Q, K, V and
// dO: a training step at B=256 H=2 L=200 d=32 fp32 75.1 -> 74.0 us, in bf16 without a causal mask 73.9 -> 72.9, B=2048 H=8 d=16 940 -> 930,
// per position at d=8 902 -> 897, B=32 H=8 L=2000 d=8 242.2 -> 240.3.  Small calls, whose branch outputs the caches would hold until
// the backward reads them, take no longer either (through / past the caches): B=4 H=8 L=100 d=16 25.3 / 25.3, B=16 H=2 L=200 d=32 52.3 / 52.3, B=32
// H=8 L=200 d=8 35.4 / 35.5, B=64 H=8 L=100 d=16 40.2 / 39.6; the largest losses of 26 shapes from B=4 to 128 were 0.5 % (per position, B=64 L=150
// 72.4 / 72.7) and 0.4 % (bf16, B=128 H=2 L=200 d=32 44.5 / 44.7).
template <typename T, int D, bool ONCE = false>
__device__ __forceinline__ void store_row4(T *dst_row, const f32x4 (&a)[Geo<D>::NMB], int g)
{
#pragma unroll
  for (int mb = 0; mb < Geo<D>::NMB; ++mb)
    if (16 * mb + 4 * g < D) {
      const float v[4] = {a[mb][0], a[mb][1], a[mb][2], a[mb][3]};
      if constexpr (ONCE) store4_once(dst_row + 16 * mb + 4 * g, v);
      else store4(dst_row + 16 * mb + 4 * g, v);
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
      store4_once(dst_row + 16 * mb + 4 * g, v);
    }
}

// zeros for the `count` elements from dst on, by one wavefront (whole rows: a multiple of 8 elements, 16-byte aligned)
template <typename T>
__device__ __forceinline__ void zero_fill(T *dst, int count, int lane)
{
  uint4 *q = reinterpret_cast<uint4 *>(dst);
  const int pieces = count * (int)sizeof(T) / 16;
  for (int i = lane; i < pieces; i += 64) q[i] = make_uint4(0u, 0u, 0u, 0u);
}
// the same by lanes `from`, `from` + `step` ...
template <typename T>
__device__ __forceinline__ void zero_rows_from(T *dst, int count, int from, int step)
{
  uint4 *q = reinterpret_cast<uint4 *>(dst);
  const int pieces = count * (int)sizeof(T) / 16;
  for (int i = from; i < pieces; i += step) q[i] = make_uint4(0u, 0u, 0u, 0u);
}

__device__ __forceinline__ unsigned abs_diff(int a, int b)  // both non-negative
{
  unsigned d;
  asm("v_sad_u32 %0, %1, %2, 0" : "=v"(d) : "v"(a), "v"(b));
  return d;
}

// mask block of position pos + r (Eq. 15): (pos + r + 1/2) / sblk, exact in fp32 while positions stay below 2^22 (the
// quotient is at least 1/(2 sblk) away from a whole number); all zero without Eq. 15, where no two blocks are then
// a power of two apart
__device__ __forceinline__ int mask_block(const KParams &p, int pos, int r = 0)
{
  return (int)fmaf((float)pos, p.sblk_inv, ((float)r + 0.5f) * p.sblk_inv);
}

// Mask block 1: the first power of two of tiles beyond the tiles that hold a key of the window.  From there on a tile at such a
// distance shows each row one key, the one at its own offset (`diagonals`).
__device__ __forceinline__ int first_diagonal(const KParams &p) { return 2 << (31 - __clz(max((p.w + kTile - 2) / kTile, 1))); }

// short-term visibility of (query i, key j + r) that the causal and validity tests let through (those make the difference
// non-negative in the causal form, so its absolute value serves both forms); plain bit operations, no branches.
__device__ __forceinline__ bool st_sees(const KParams &p, int i, int j, int kid_i, int kid_j, bool last)
{
  return (abs_diff(i, j) < (unsigned)p.w) | (__popc(abs_diff(kid_i, kid_j)) == 1) | last;
}

// Four bits a lane: which of the elements 4g .. 4g+3 of a tile its own row sees.  Without Eq. 15, or with its mask block 1,
// visibility is a function of the distance alone, own - element = 16*dt + c - r with dt tiles between the two and c = q - 4g: the
// bits of the tiles next to the row's own (dt of 0, 1 and -1) are cut out of one table over distances, once per wavefront.
// Powers of two from first_diagonal on are left to `diagonals`.  A general tile of the forward takes 35 vector instructions for its
// masks and sums, 69 with a test per element.  (Larger mask blocks are tested element by element, and no table is made: selection +
// forward at B=40 H=8 L=87 d=16 bf16 with mask block 16, in both directions, 16.6 us with it, 16.3 without.)
struct LaneMasks {
  int c;
  unsigned near;  // bits 0-3, 4-7, 8-11: dt = 0, 1, -1 (the window and the powers of two of Eq. 15)
  __device__ __forceinline__ static LaneMasks make(const KParams &p, int q, int g)
  {
    LaneMasks m{};
    if (p.sblk > 1) return m;
    m.c = q - 4 * g;
    unsigned long long table = p.w >= 32 ? ~0ull : ((1ull << (2 * p.w - 1)) - 1) << (33 - p.w);  // bit 32 + distance
    if (p.sblk == 1) table |= 0x0001011600000000ull | 0x00000000D1010000ull;  // 1, 2, 4, 8, 16 on either side
    auto cut = [&](int x) { return (unsigned)(table >> (32 - x)) & 15u; };  // element r at distance x - r, the table being symmetric
    m.near = cut(m.c) | cut(m.c + kTile) << 4 | cut(m.c - kTile) << 8;
    return m;
  }
  // elements from x on; elements below x (x counted from the first of the four)
  __device__ __forceinline__ static unsigned from(int x) { return 15u << clamp4(x); }
  __device__ __forceinline__ static unsigned below(int x) { return 15u >> (4 - clamp4(x)); }
  __device__ __forceinline__ static int clamp4(int x) { return min(max(x, 0), 4); }
  // of the keys from key0 on, those that the causal and validity tests let query row i see
  __device__ __forceinline__ static unsigned keys(const KParams &p, int key0, int p0, int i)
  {
    return from(p0 - key0) & below((p.bidir ? p.L : i + 1) - key0);
  }
  // FAR: those too
  template <bool FAR = false>
  __device__ __forceinline__ unsigned st(const KParams &p, int dt) const
  {
    const int far = dt < 0 ? -dt : dt;
    if (far <= 1) return near >> (dt == 0 ? 0 : dt == 1 ? 4 : 8);
    const int d0 = kTile * dt + c;
    unsigned m = from(d0 - p.w + 1) & below(d0 + p.w);
    if (p.sblk == 1 && (far & (far - 1)) == 0 && (FAR || far < first_diagonal(p))) m |= from(c) & below(c + 1);
    return m;
  }
};
// x where bit r is set, else zero (of a NaN too)
__device__ __forceinline__ float keep(float x, unsigned bits, int r)
{
  return __uint_as_float(__float_as_uint(x) & (unsigned)__builtin_amdgcn_sbfe((int)bits, r, 1));
}

// THE NEAR FORM: causal, without Eq. 15 or with its mask block 1, and a window that ends within the tile before the row's own (w <= 17).
// The short-term branch is then the row's own tile, the one before and the diagonals; every mask of those two tiles is the same
// for all tiles of a wavefront, and is kept as four scalars, one per element of a lane (bit l: lane l's element r): a masked element
// costs one v_cndmask on a scalar pair, and what tiles combine (padding, the tile's own triangle, whether it is selected) is scalar work.
// The two tiles of the forward's short-term branch take 54 vector instructions, 125 with masks as bits.
typedef unsigned long long Word;
__host__ __device__ __forceinline__ bool near_form(const KParams &p) { return p.bidir == 0 && p.sblk <= 1 && p.w <= kTile + 1; }
__device__ __forceinline__ bool in_lanes(Word m) { return __builtin_amdgcn_inverse_ballot_w64(m); }
// the lanes (q, g) with 4g + r <= q, and with 4g + r >= q
constexpr Word triangle(int r, bool upper)
{
  Word m = 0;
  for (int l = 0; l < 64; ++l)
    if (upper ? 4 * (l >> 4) + r >= (l & 15) : 4 * (l >> 4) + r <= (l & 15)) m |= 1ull << l;
  return m;
}
// the lanes with 4g + r >= x (0 <= x <= 16)
__device__ __forceinline__ Word elements_from(int x, int r)
{
  const int n = 16 * ((x - r + 3) >> 2);
  return n >= 64 ? 0ull : ~0ull << n;
}
inline NearMasks near_masks(const KParams &p, bool key_side) { return NearMasks(p.w, p.sblk == 1, key_side); }

// may any query of tile I see any key of tile J in the short-term branch (J <= I in the causal form)?
__device__ __forceinline__ bool st_reaches(const KParams &p, int I, int J)
{
  const int hi = max(I, J) * kTile, lo = min(I, J) * kTile;
  const bool window = hi - lo - (kTile - 1) < p.w;
  if (p.sblk == 0) return window;
  // largest mask-block distance of the two tiles' positions, and the largest power of two in it, against the smallest
  const int top = mask_block(p, hi, kTile - 1) - mask_block(p, lo);
  const int bottom = mask_block(p, hi) - mask_block(p, lo, kTile - 1);
  const int pow2 = 1 << (31 - __clz(top | 1));
  return window | ((top >= 1) & (pow2 >= bottom)) | (J * kTile + kTile - 1 >= p.last_lo);
}

// A tensor slice behind a buffer descriptor: loads take 32-bit byte offsets (no address arithmetic in vector registers)
// and return zeros past the end of the slice, which is how the rows of the last, partial tile read.
constexpr unsigned kNowhere = 0xFFFFF000u;  // a byte offset past every slice
struct Slice {
  __amdgpu_buffer_rsrc_t d;
  __device__ __forceinline__ Slice(const void *base, size_t bytes)
      : d(__builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes, 0x00027000)) {}
};
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
template <typename T, int N>
__device__ __forceinline__ void load_n(const Slice &s, unsigned off, float (&o)[N])
{
  if constexpr (sizeof(T) == 4) {
    if constexpr (N == 2) {
      const u32x2_t v = __builtin_amdgcn_raw_buffer_load_b64(s.d, off, 0, 0);
      o[0] = __uint_as_float(v[0]); o[1] = __uint_as_float(v[1]);
    } else {
#pragma unroll
      for (int i = 0; i < N; i += 4) {
        const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(s.d, off + 4 * i, 0, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) o[i + e] = __uint_as_float(v[e]);
      }
    }
  } else {
    unsigned w[N / 2];
    if constexpr (N == 2) {
      w[0] = __builtin_amdgcn_raw_buffer_load_b32(s.d, off, 0, 0);
    } else if constexpr (N == 4) {
      const u32x2_t v = __builtin_amdgcn_raw_buffer_load_b64(s.d, off, 0, 0);
      w[0] = v[0]; w[1] = v[1];
    } else {
      const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(s.d, off, 0, 0);
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = v[e];
    }
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
      o[2 * i] = __uint_as_float(w[i] << 16);
      o[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
    }
  }
}

// N bytes' worth of registers as they stand
template <int N>
__device__ __forceinline__ void load_raw(const Slice &s, unsigned off, unsigned (&w)[N])
{
  if constexpr (N == 1) {
    w[0] = __builtin_amdgcn_raw_buffer_load_b32(s.d, off, 0, 0);
  } else if constexpr (N == 2) {
    const u32x2_t v = __builtin_amdgcn_raw_buffer_load_b64(s.d, off, 0, 0);
    w[0] = v[0]; w[1] = v[1];
  } else {
    const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(s.d, off, 0, 0);
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = v[e];
  }
}
template <typename T, int D>
__device__ __forceinline__ void load_op(const Slice &s, unsigned off, typename Operands<T, D>::Row &o)
{
  if constexpr (Operands<T, D>::kBf) load_raw(s, off, o.w);
  else load_n<T>(s, off, o.v);
}

// The lane id, rebuilt where it stands: addresses formed from it are not computed ahead of a walk and kept in registers
// through it.
__device__ __forceinline__ int fresh_lane()
{
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}

// one head's [L,D] rows as matrix operands
template <typename T, int D>
struct Rows {
  static constexpr bool kNear = false;  // far: operands are requested a tile ahead
  static constexpr unsigned TB = kTile * D * sizeof(T);  // bytes of a tile
  Slice s;
  unsigned row_off, col_off, own_off;  // this lane's place in a tile
  __device__ __forceinline__ Rows(const T *head, int L, int q, int g) : s(head, (size_t)L * D * sizeof(T))
  {
    row_off = (unsigned)(q * D + Geo<D>::CPL * g) * (unsigned)sizeof(T);
    own_off = (unsigned)(q * D + (D == 8 ? 0 : (4 * g) & (D - 1))) * (unsigned)sizeof(T);
    col_off = (unsigned)(4 * g * D + (D < 16 ? (q & (D - 1)) : q)) * (unsigned)sizeof(T);
  }
  // contraction over channels: channels CPL*g .. of row q of tile t
  __device__ __forceinline__ void op(int t, typename Operands<T, D>::Row &o) const { load_op<T, D>(s, row_off + (unsigned)t * TB, o); }
  __device__ __forceinline__ void row(int t, float (&o)[Geo<D>::CPL]) const { load_n<T>(s, row_off + (unsigned)t * TB, o); }
  // contraction over the tile's rows: element r is row 4g + r, channel 16*mb + q (d = 8: lanes q and q + 8 hold the same)
  __device__ __forceinline__ void col(int t, typename Operands<T, D>::Col (&o)[Geo<D>::NMB]) const
  {
    const unsigned off = col_off + (unsigned)t * TB;
#pragma unroll
    for (int mb = 0; mb < Geo<D>::NMB; ++mb) {
      unsigned x[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const unsigned at = off + (unsigned)((r * D + 16 * mb) * sizeof(T));
        if constexpr (sizeof(T) == 4) x[r] = __builtin_amdgcn_raw_buffer_load_b32(s.d, at, 0, 0);
        else x[r] = (unsigned)__builtin_amdgcn_raw_buffer_load_b16(s.d, at, 0, 0);
      }
      if constexpr (Operands<T, D>::kBfCol) {
        o[mb].w[0] = x[0] | x[1] << 16;
        o[mb].w[1] = x[2] | x[3] << 16;
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) o[mb].v[r] = __uint_as_float(sizeof(T) == 4 ? x[r] : x[r] << 16);
      }
    }
  }
  // all eight channels of row q (d = 8)
  __device__ __forceinline__ void whole(int t, float (&o)[D]) const { load_n<T>(s, own_off + (unsigned)t * TB, o); }
  // row q of the tile, the channels of this lane's accumulators: element r is channel 16*mb + 4g + r
  __device__ __forceinline__ void own(int t, float (&o)[Geo<D>::NMB][4]) const
  {
#pragma unroll
    for (int mb = 0; mb < Geo<D>::NMB; ++mb) load_n<T>(s, own_off + (unsigned)t * TB + 16u * mb * (unsigned)sizeof(T), o[mb]);
  }
};

template <int N>
__device__ __forceinline__ void store_lds(float *p, const float (&o)[N])
{
  if constexpr (N == 2) {
    *reinterpret_cast<float2 *>(p) = make_float2(o[0], o[1]);
  } else {
#pragma unroll
    for (int i = 0; i < N; i += 4) *reinterpret_cast<float4 *>(p + i) = make_float4(o[i], o[i + 1], o[i + 2], o[i + 3]);
  }
}
// the same from LDS, where a workgroup staged the head: fp32 rows of D + 4 floats (20 or 36; d = 8: 8), or the bf16 bits themselves in
// rows of D + 4 (d = 16) or D + 8 halfwords; rows stay aligned for a row operand's load.  Of the LDS' index cycles bank conflicts take
// a quarter at d = 32 in fp32, a third there in bf16 and at d = 16, and at d = 8, whose rows q and q + 8 share their banks, half in the forward
// and two fifths in the backward (profiles/small_heads_pipe_counters.txt); the LDS is busy 4 to 22 % of the time.  Without conflicts cost
// more: d = 8 in rows of 12, three backward workgroups per CU where the registers allow four, positions at B=2048 L=200 635 us, 569
// so; the 16-byte halves of rows q >= 8 swapped, two fifths of the conflicts less and the whole of it 1-3 % slower.
// In floats; the kernels lay their LDS out with it, the launches size it.
constexpr int lds_row(bool bf16, int d) { return stored_bits(bf16, d) ? (d == 32 ? 20 : 10) : d == 8 ? 8 : d + 4; }
template <typename T, int D>
constexpr int kLdsRow = lds_row(std::is_same<T, bf16_t>::value, D);
template <typename T, int D>
struct LdsRows {
  static constexpr bool kNear = true;  // near: operands are read where they are used and take no registers before
  static constexpr bool kBf = Operands<T, D>::kBf;
  static constexpr int R = kLdsRow<T, D>, NMB = Geo<D>::NMB, CPL = Geo<D>::CPL;
  const float *row_at, *col_at, *own_at;  // this lane's place in tile 0
  __device__ __forceinline__ LdsRows(const float *base, int q, int g)
  {
    if constexpr (kBf) {  // (col: the transposing read takes rows 4g .. 4g+3, 16 channels of them spread over 16 lanes)
      row_at = base + q * R + CPL / 2 * g;
      col_at = base + (4 * g + (q >> 2)) * R + 2 * (q & 3);
      own_at = base + q * R + 2 * g;
    } else {
      row_at = base + q * R + CPL * g;
      col_at = base + 4 * g * R + (D < 16 ? (q & (D - 1)) : q);
      own_at = base + q * R + (D == 8 ? 0 : 4 * g & (D - 1));
    }
  }
  __device__ __forceinline__ void op(int t, typename Operands<T, D>::Row &o) const
  {
    const float *at = row_at + t * (kTile * R);
    if constexpr (kBf && D == 32) {
      const uint4 v = *reinterpret_cast<const uint4 *>(at);
      o.w[0] = v.x; o.w[1] = v.y; o.w[2] = v.z; o.w[3] = v.w;
    } else if constexpr (kBf) {
      const uint2 v = *reinterpret_cast<const uint2 *>(at);
      o.w[0] = v.x; o.w[1] = v.y;
    } else {
      load_n<CPL>(at, o.v);
    }
  }
  __device__ __forceinline__ void row(int t, float (&o)[CPL]) const
  {
    typename Operands<T, D>::Row x;
    op(t, x);
    Operands<T, D>::floats(x, o);
  }
  __device__ __forceinline__ void col(int t, typename Operands<T, D>::Col (&o)[NMB]) const
  {
    const float *at = col_at + t * (kTile * R);
#pragma unroll
    for (int mb = 0; mb < NMB; ++mb) {
      if constexpr (kBf) {
        const u32x2_t v = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((mfma::lds_s16x4 *)(at + 8 * mb)));
        if constexpr (Operands<T, D>::kBfCol) {
          o[mb].w[0] = v[0]; o[mb].w[1] = v[1];
        } else {
          o[mb].v[0] = __uint_as_float(v[0] << 16);
          o[mb].v[1] = __uint_as_float(v[0] & 0xFFFF0000u);
          o[mb].v[2] = __uint_as_float(v[1] << 16);
          o[mb].v[3] = __uint_as_float(v[1] & 0xFFFF0000u);
        }
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) o[mb].v[r] = at[r * R + 16 * mb];
      }
    }
  }
  __device__ __forceinline__ void whole(int t, float (&o)[D]) const { load_n<D>(own_at + t * (kTile * R), o); }
  __device__ __forceinline__ void own(int t, float (&o)[NMB][4]) const
  {
#pragma unroll
    for (int mb = 0; mb < NMB; ++mb) {
      const float *at = own_at + t * (kTile * R) + (kBf ? 8 : 16) * mb;
      if constexpr (kBf) load4(reinterpret_cast<const bf16_t *>(at), o[mb]);
      else load_n<4>(at, o[mb]);
    }
  }
  // where a row's operand stands: `base` as above
  static __device__ __forceinline__ void put(float *base, int row, int g, const typename Operands<T, D>::Row &x)
  {
    float *at = base + row * R + (kBf ? CPL / 2 : CPL) * g;
    if constexpr (kBf && D == 32) *reinterpret_cast<uint4 *>(at) = make_uint4(x.w[0], x.w[1], x.w[2], x.w[3]);
    else if constexpr (kBf) *reinterpret_cast<uint2 *>(at) = make_uint2(x.w[0], x.w[1]);
    else store_lds(at, x.v);
  }
};
// two heads' rows from tile T0 on into LDS; rows before p0 (the padding) and past the end are zeros.  CLEAN: elements that are
// not finite become zeros too.  A wavefront requests N of its tiles before it waits for the first.
// between(): called once, by every wavefront, after the first requests and before the first row is written.
template <int D>
constexpr int kStageAhead = D == 32 ? 2 : 4;
struct Nothing {
  __device__ __forceinline__ void operator()() const {}
};
template <typename T, int D, bool CLEAN, int N = 1, typename Between = Nothing>
__device__ __forceinline__ void stage_pair(const T *A, const T *B, float *a_lds, float *b_lds, int L, int T0, int NT, int p0, int lane, int wv,
                                           int W, Between &&between = {})
{
  const int q = lane & 15, g = lane >> 4;
  const Rows<T, D> Ar(A, L, q, g), Br(B, L, q, g);
  if (T0 + wv >= NT) between();
  for (int t0 = T0 + wv; t0 < NT; t0 += N * W) {
    typename Operands<T, D>::Row x[N], y[N];
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const int t = t0 + n * W;
      const unsigned off = (t < NT) & (t * kTile + q >= p0) ? Ar.row_off + (unsigned)t * Rows<T, D>::TB : kNowhere;
      load_op<T, D>(Ar.s, off, x[n]);
      load_op<T, D>(Br.s, off, y[n]);
    }
    if constexpr (N > 1) asm volatile("" ::: "memory");  // (the requests are not moved to where their rows are used)
    if (t0 == T0 + wv) between();
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const int t = t0 + n * W;
      if (t >= NT) break;
      if constexpr (CLEAN) {
        Operands<T, D>::clean(x[n]);
        Operands<T, D>::clean(y[n]);
      }
      LdsRows<T, D>::put(a_lds, t * kTile + q, g, x[n]);
      LdsRows<T, D>::put(b_lds, t * kTile + q, g, y[n]);
    }
  }
}

// pairs of bits (blocks of 8) -> one bit per tile
__device__ __forceinline__ unsigned pair_bits(unsigned long long b)
{
  b = (b | (b >> 1)) & 0x5555555555555555ull;
  b = (b | (b >> 1)) & 0x3333333333333333ull;
  b = (b | (b >> 2)) & 0x0F0F0F0F0F0F0F0Full;
  b = (b | (b >> 4)) & 0x00FF00FF00FF00FFull;
  b = (b | (b >> 8)) & 0x0000FFFF0000FFFFull;
  return (unsigned)(b | (b >> 16));
}

// THE WALK.  Tiles are grouped by kind, 64 tiles (a word) at a time, as three bit masks in scalar registers, and each kind
// has a loop of its own whose body is one straight line: no branches, so the accumulators stay in place and the loads of the
// next tile (of whatever kind) are waited for where they are used.
//   0 general   both branches, every mask test: tiles of both branches, the diagonal, the first and the last valid tile, and
//               tiles with last-block keys of Eq. 15
//   1 lt        long-term only: no mask (per-element selection tests where blocks are smaller than tiles or per position)
//   2 st        short-term only: window and power-of-two tests
// A lane classifies a tile, ballots make the words: about 20 instructions, where bit arithmetic on scalars took over a hundred
// for half as many tiles and the scalar ALU was as busy as the vector ALUs (with the masks as bits, the steps above: 289 and 956 us).
struct Walk {
  Word m0 = 0, m1 = 0, m2 = 0;  // tiles of the word still to come
  Word lt = 0;                  // long-term tiles of the word
  int base = 0;                 // first tile of the word
  // Word w of the walk of tile X (a query tile when KEY_SIDE is false, else a key tile) over the tiles lo .. hi.  lt_here: the
  // long-term branch takes the lane's tile.  edge: the lane's tile needs every test.  dia: also the short-term tiles that
  // `diagonals` takes, for a walk that leaves it out.  with_st: there is a short-term branch.  ST_GENERAL: every short-term tile
  // needs every test (long-term ones beyond its reach do not: forward at B=19 H=8 L=155 d=32 b=8 13.6 us with them, 12.6 without).
  template <bool KEY_SIDE, bool ST_GENERAL = false>
  __device__ __forceinline__ void start(const KParams &p, int X, int w, int lo, int hi, int lane, bool lt_here, bool edge, bool dia,
                                        bool with_st)
  {
    base = w * 64;
    const int t = base + lane;
    const bool in = (unsigned)(t - lo) <= (unsigned)(hi - lo);
    bool st;
    if (p.sblk > 1) {
      st = KEY_SIDE ? st_reaches(p, t, X) : st_reaches(p, X, t);
    } else {
      const int reach = max((p.w + kTile - 2) / kTile, p.sblk);  // tiles up to this far away hold a key of the window, or the next power of two
      st = abs_diff(t, X) <= (unsigned)reach;
      if (p.sblk == 1) {
        if (dia) st |= __popc(abs_diff(t, X)) == 1;
        // the last position: its tile is walked by every query tile (that reaches it)
        st |= (KEY_SIDE ? X : t) >= p.last_lo / kTile;
      }
    }
    st &= with_st;
    lt = __ballot(in & lt_here);
    const Word s = __ballot(in & st), e = __ballot(edge);
    m0 = ST_GENERAL ? s | (e & lt) : (lt & s) | (e & (lt | s));
    m1 = lt & ~m0;
    m2 = s & ~lt & ~m0;
  }
  __device__ __forceinline__ Word all() const { return m0 | m1 | m2; }
  __device__ __forceinline__ static int first(Word m) { return __builtin_ctzll(m); }
  // the first tile still to come (some tile when there is none: a harmless read-ahead)
  __device__ __forceinline__ int peek() const
  {
    const Word m = m0 ? m0 : m1 ? m1 : m2;
    return base + (m ? first(m) : 0);
  }
  __device__ __forceinline__ int take(Word &m) const
  {
    const int t = base + first(m);
    m &= m - 1;
    return t;
  }
  __device__ __forceinline__ bool is_lt(int t) const { return (lt >> (t & 63)) & 1ull; }
};

// THE DIAGONALS of mask block 1.  A row sees one key of a tile 2, 4, 8 ... tiles away (from first_diagonal on), its own offset's:
// 16 pairs, for which a matrix product would form 256.  They are taken four distances at a time on the vector ALUs instead: every
// lane multiplies its channels of its row for all four distances (d = 8: see add_row), gather_g leaves distance n's sum with lane group n, where the
// mask and the exponential are, and spread_g hands the four results to all groups, which add them into their accumulators'
// channels (`own`).  About 12 vector instructions a distance; as tiles of the walk the distances took half of its steps at L=2000
// (a training step at B=32 H=8 L=2000 d=8 356 us, 302 like this; B=2048 H=8 L=200 d=16 1050 and 996).
// They come after the walk: they may then use its registers (ahead of it d = 32 and the forward at d = 8 spilled), and the walk's sums are
// not rounded at the size of these large terms (dQ at L=450 d=16 against 64 bits: ahead 1.028 times the error that tiles had, so
// 1.014; the rest is the rounding of products on the vector ALUs, and the lse more than makes up for it, see the forward).
// First they are where that is better: the forward of bf16 rows at d = 32, whose walk adds with fewer roundings (o_st at L=1000: 1.04 of
// the error after it) and has the registers; the backward at d = 8, whose sums are a lane group's own parts and whose walk runs 2 %
// faster so (L=1657: 69.0 and 70.3 us).
// f(d): tiles X + d, X + 2d, X + 4d, X + 8d (some may lie outside lo .. hi: d times the lane group's power tells).
template <typename F>
__device__ __forceinline__ void diagonals(const KParams &p, int X, int lo, int hi, F &&f)
{
  const int d0 = first_diagonal(p);
  for (int d = d0; d <= X - lo; d <<= 4) f(-d);
  for (int d = d0; d <= hi - X; d <<= 4) f(d);
}
template <int D>
constexpr bool kFarFirst = Geo<D>::kQuads;
// The backward from d = 16 on under a selection per position leaves them in the walk: nearly every tile is walked there for some row's
// selection, and these keys cost it a mask, where a batch of distances costs the time of a tile.  Gradients with them and without, us:
// B=300 H=4 over 2 L=200 d=32 222 and 170 (204 with a tile of its own kind for a distance), B=700 H=8 over 4 L=180 d=16 289 and 275; in the
// forward they gain at d = 32 too (61.7 and 64.6).
template <int D, bool PERPOS>
constexpr bool kDiagonals = !(PERPOS && D >= 16);
// d = 32: the phases of a batch of distances are kept apart: their registers would spill
template <int D>
__device__ __forceinline__ void phase_end()
{
  if constexpr (D == 32) __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ float gather_g(const float (&x)[4])
{
  const u32x2_t a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[0]), __float_as_uint(x[1]), false, false);
  const u32x2_t b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[2]), __float_as_uint(x[3]), false, false);
  const float u = __uint_as_float(a[0]) + __uint_as_float(a[1]), v = __uint_as_float(b[0]) + __uint_as_float(b[1]);
  const u32x2_t c = __builtin_amdgcn_permlane32_swap(__float_as_uint(u), __float_as_uint(v), false, false);
  return __uint_as_float(c[0]) + __uint_as_float(c[1]);
}
__device__ __forceinline__ void spread_g(float x, float (&o)[4])
{
  const unsigned u = __float_as_uint(x);
  const u32x2_t a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const u32x2_t b = __builtin_amdgcn_permlane32_swap(a[0], a[0], false, false);
  const u32x2_t c = __builtin_amdgcn_permlane32_swap(a[1], a[1], false, false);
  o[0] = __uint_as_float(b[0]); o[1] = __uint_as_float(c[0]); o[2] = __uint_as_float(b[1]); o[3] = __uint_as_float(c[1]);
}
// d = 8: a row is two 16-byte loads, so a lane group takes a whole distance by itself and adds to its own part of the sums
// (Operands::add): nothing to gather or to spread
__device__ __forceinline__ void whole_row(const float (&x)[2], float (&o)[8])  // a row spread over the lane groups, into each of them
{
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    float y[4];
    spread_g(x[i], y);
#pragma unroll
    for (int n = 0; n < 4; ++n) o[2 * n + i] = y[n];
  }
}
__device__ __forceinline__ void add_row(f32x4 (&acc)[2], float c, const float (&a)[8])
{
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i / 4][i % 4] = fmaf(c, a[i], acc[i / 4][i % 4]);
}
template <int N>
__device__ __forceinline__ void own_of_row(const float (&x)[N], float (&o)[1][4])  // d = 16: the same channels
{
#pragma unroll
  for (int r = 0; r < 4; ++r) o[0][r] = x[r & (N - 1)];
}
// four distances' products, summed before they meet the accumulators: one rounding at their size instead of four
template <int N>
__device__ __forceinline__ void add_own(f32x4 (&acc)[N], const float (&c)[4], const float (&a)[4][N][4])
{
#pragma unroll
  for (int mb = 0; mb < N; ++mb)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[mb][r] += fmaf(c[3], a[3][mb][r], fmaf(c[2], a[2][mb][r], fmaf(c[1], a[1][mb][r], c[0] * a[0][mb][r])));
}

// What a query tile's wavefront knows about its long-term selection.  In LDS (this wavefront's words): sel rows of
// its query blocks as bits over key blocks [kTile/BK][NWb], then the tile words [NWt].  Per-position form: `row` is the
// lane's own row (at most 64 key blocks).
template <int BK, bool PERPOS>
struct LtSel {
  static constexpr int NROW = PERPOS ? 0 : kTile / BK;
  unsigned *bits, *tiles;
  int NWb;
  unsigned long long row, all;  // (per position: and the tiles that any of the rows selected)

  // sel rows: of query block x0 on, or, per position, of this lane's position (which may take no part).  p0: the
  // first valid position.  Entries outside [0, NB), later blocks (causal form) and blocks without a valid key drop out.
  // `first`: the entries as `request` fetched them, per position the first four of this lane's row, else entry e in lane e
  static constexpr int kFirst = PERPOS ? 4 : 1;
  static __device__ __forceinline__ void request(const KParams &p, const int *sel_head, int I, int iq, int lane, int (&first)[kFirst])
  {
    if constexpr (PERPOS) {
      const int *row = sel_head + (size_t)min(iq, p.L - 1) * p.k;
#pragma unroll
      for (int i = 0; i < 4; ++i) first[i] = row[min(i, p.k - 1)];
    } else {
      const int rows = min(NROW, p.NB - I * NROW);  // (two blocks to a tile: the last tile may have one)
      first[0] = sel_head[(size_t)I * NROW * p.k + min(lane, rows * p.k - 1)];
    }
  }
  __device__ __forceinline__ void build(const KParams &p, unsigned *lds, const int *sel_rows, const int *sel_pos, bool takes_part, int I,
                                        int iq, int p0, int lane, const int (&first)[kFirst])
  {
    NWb = (p.NB + 31) / 32;
    const int NWt = ((p.L + kTile - 1) / kTile + 31) / 32;
    bits = lds;
    tiles = lds + NROW * NWb;
    row = all = 0ull;
    if constexpr (PERPOS) {
      // (later blocks and blocks without a valid key may stay: no walk asks about their tiles; with two blocks to a tile it does)
      auto taken = [&](int J) { return (unsigned)J < (unsigned)p.NB && (BK == kTile || (J * BK <= iq && (J + 1) * BK > p0)); };
      const bool half = p.NB <= 32;
      auto add = [&](const int (&J)[4]) __attribute__((always_inline)) {
        if (half) {
          unsigned x = 0u;
#pragma unroll
          for (int i = 0; i < 4; ++i) x |= taken(J[i]) ? 1u << J[i] : 0u;
          row |= x;
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) row |= taken(J[i]) ? 1ull << J[i] : 0ull;
        }
      };
      add(first);  // (apart from the others: a load in the loop, though never issued, would have this wait for all that are on their way)
      // four requests at a time: a loop of single ones waited for memory k times (B=2048 H=8 over 4 L=200 d=8: 1093 us, 1060 so)
      for (int e = 4; e < p.k; e += 4) {
        int J[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) J[i] = sel_pos[min(e + i, p.k - 1)];
        add(J);
      }
      if (!takes_part) row = 0ull;
      all = (unsigned)__builtin_amdgcn_readfirstlane(or_row((unsigned)row));
      if (!half) all |= (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane(or_row((unsigned)(row >> 32))) << 32;
      if (BK < kTile) all = pair_bits(all);
      if (lane < NWt) tiles[lane] = lane == 0 ? (unsigned)all : (unsigned)(all >> 32);
    } else {
      for (int i = lane; i < NROW * NWb + NWt; i += 64) bits[i] = 0u;
      auto add = [&](int i, int J) __attribute__((always_inline)) {
        const int xr = NROW == 1 ? 0 : (i >= p.k ? 1 : 0);
        const int x = I * NROW + xr;
        if (i >= NROW * p.k || x >= p.NB || J < 0 || J >= p.NB || (J > x && !p.bidir) || (J + 1) * BK <= p0) return;
        atomicOr(&bits[xr * NWb + (J >> 5)], 1u << (J & 31));
        const int t = J * BK / kTile;
        atomicOr(&tiles[t >> 5], 1u << (t & 31));
      };
      add(lane, first[0]);  // (consecutive rows are contiguous)
      const int count = min(NROW, p.NB - I * NROW) * p.k;
      for (int i = lane + 64; i < count; i += 64) add(i, sel_rows[i]);
    }
  }
  // the same where nothing was requested ahead (per block): entries kept from before this point cost the longer walks registers, 1 % of
  // a training step without a causal mask at B=132 H=8 L=70 d=8
  __device__ __forceinline__ void build(const KParams &p, unsigned *lds, const int *sel_rows, int I, int p0, int lane)
  {
    static_assert(!PERPOS, "a row per block");
    NWb = (p.NB + 31) / 32;
    const int NWt = ((p.L + kTile - 1) / kTile + 31) / 32;
    bits = lds;
    tiles = lds + NROW * NWb;
    row = all = 0ull;
    for (int i = lane; i < NROW * NWb + NWt; i += 64) bits[i] = 0u;
    for (int i = lane; i < NROW * p.k; i += 64) {
      const int xr = NROW == 1 ? 0 : (i >= p.k ? 1 : 0);
      const int x = I * NROW + xr;
      if (x >= p.NB) continue;
      const int J = sel_rows[i];  // (consecutive rows are contiguous)
      if (J < 0 || J >= p.NB || (J > x && !p.bidir) || (J + 1) * BK <= p0) continue;
      atomicOr(&bits[xr * NWb + (J >> 5)], 1u << (J & 31));
      const int t = J * BK / kTile;
      atomicOr(&tiles[t >> 5], 1u << (t & 31));
    }
  }
  static __device__ __forceinline__ unsigned or_row(unsigned x)
  {
    x |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xf, 0xf, false);
    x |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x124, 0xf, 0xf, false);
    x |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x122, 0xf, 0xf, false);
    return x | (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x121, 0xf, 0xf, false);
  }
  __device__ __forceinline__ bool has_tile(int t) const { return (tiles[t >> 5] >> (t & 31)) & 1u; }
  // did the lane's row select the block of its keys (four keys from key0 on share one)?  Only asked about tiles in `tiles`.
  __device__ __forceinline__ bool sees(int q, int key0) const
  {
    const int Jb = key0 / BK;
    if constexpr (PERPOS) return (row >> Jb) & 1ull;
    else if constexpr (BK < kTile) return (bits[(q / BK) * NWb + (Jb >> 5)] >> (Jb & 31)) & 1u;
    else return true;
  }
};
// the OR over the wavefront
__device__ __forceinline__ unsigned or_all(unsigned x)
{
  x = LtSel<kTile, true>::or_row(x);
  u32x2_t a = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  const unsigned y = a[0] | a[1];
  a = __builtin_amdgcn_permlane32_swap(y, y, false, false);
  return __builtin_amdgcn_readfirstlane(a[0] | a[1]);
}
// the same of a tile of the near form with one block to a tile: the entries stay in registers, 64 at a time, lane e holding entry e
struct PickedTiles {
  const int *rows;
  int k, J;
  // tiles 64w .. 64w + 63, whatever else the entries name: every lane's bit, and their OR over the wavefront.  (Entry by entry, six scalar
  // instructions each, a step at B=2 H=2 L=600 d=16 took 40.6 us with lists of 9 and 60.0 with lists of 35; 39.7 and 57.7 so, of 4 the same.)
  __device__ __forceinline__ Word word(int w, int lane) const
  {
    Word m = 0;
    auto add = [&](int x, int count) __attribute__((always_inline)) { m |= (x >> 6) == w && lane < count ? 1ull << (x & 63) : 0ull; };
    add(J, k);  // (apart from the others: a load in the loop, though never issued, would have this wait for all that are on their way)
    for (int e0 = 64; e0 < k; e0 += 64) add(rows[min(e0 + lane, k - 1)], k - e0);
    return (Word)or_all((unsigned)(m >> 32)) << 32 | or_all((unsigned)m);
  }
};
__host__ __device__ inline int lt_words(const KParams &p, bool perpos)
{
  return (perpos ? 0 : kTile / p.b) * ((p.NB + 31) / 32) + ((p.L + kTile - 1) / kTile + 31) / 32;
}


// HEADS BY LENGTH.  A few heads to a CU: the launch lasts as long as the fullest CU, and which lengths meet there was chance.  The
// workgroups therefore take the units (heads, or groups) in the order of their rows' lengths, the longest first; where all are there
// from the start, two to a CU, the second of them the other way round: the longest beside the shortest.  One wavefront of a workgroup
// finds the place: it holds all lengths (64 to a register), settles two bits at a time the length that stands at its rank and takes the
// row among those of that length, ties by index.  Lengths that differ by less than an eighth of the longest stay in turn (beyond a quarter they never do).
constexpr int kOrderRows = 512;
constexpr int kCUs = 256;
struct Unit {
  int id, valid;  // and the length of its row
};
__device__ __forceinline__ Unit unit_by_length(const int *valid_len, const KParams &p, int per_row, unsigned pid, unsigned units)
{
  constexpr int N = kOrderRows / 64;
  const int lane = threadIdx.x & 63;
  const int in_turn = clamp_len(valid_len[pid / per_row], p.L);  // (beside the other loads, not after them)
  int len[N];
  // f(i) for the registers that hold rows, four at a time
  auto each = [&](auto f) __attribute__((always_inline)) {
#pragma unroll
    for (int i0 = 0; i0 < N; i0 += 4)
      if (i0 == 0 || 64 * i0 < p.B)
#pragma unroll
        for (int i = i0; i < i0 + 4; ++i) f(i);
  };
#pragma unroll
  for (int i = 0; i < N; ++i) len[i] = -1;
  each([&](int i) { len[i] = valid_len[min(64 * i + lane, p.B - 1)]; });
  int longest = 0, shortest = p.L;
  each([&](int i) {
    len[i] = clamp_len(len[i], p.L);
    longest = max(longest, len[i]);
    shortest = min(shortest, len[i]);
    if (64 * i + lane >= p.B) len[i] = -1;
  });
  // (every lane's lengths with those of lane 0)
  longest = max(longest, __builtin_amdgcn_readfirstlane(longest));
  shortest = min(shortest, __builtin_amdgcn_readfirstlane(shortest));
  if (__ballot(8 * (longest - shortest) >= longest) == 0ull) return {(int)pid, in_turn};
  const unsigned place = pid >= kCUs && units <= 2 * kCUs ? units - 1 - (pid - kCUs) : pid;
  const int rank = (int)place / per_row;
  // the largest length that more than `rank` rows reach, two bits at a time
  int x = 0;
  for (int bit = (31 - __builtin_clz((unsigned)p.L)) & ~1; bit >= 0; bit -= 2) {
    int c[3] = {0, 0, 0};
    each([&](int i) {
#pragma unroll
      for (int n = 0; n < 3; ++n) c[n] += __popcll(__ballot(len[i] >= (x | (n + 1) << bit)));
    });
    x |= ((c[0] > rank) + (c[1] > rank) + (c[2] > rank)) << bit;
  }
  int left = rank, row = 0;
  each([&](int i) { left -= __popcll(__ballot(len[i] > x)); });
  each([&](int i) {
    const unsigned long long m = __ballot(len[i] == x);
    const int n = __popcll(m), before = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
    if (left >= 0 && left < n) row = 64 * i + __builtin_ctzll(__ballot(len[i] == x && before == left));
    left -= n;
  });
  return {row * per_row + (int)place % per_row, x};
}
// the unit of this workgroup, the same in all of its wavefronts
__device__ __forceinline__ Unit place_by_length(const int *valid_len, const KParams &p, int per_row, int wv)
{
  __shared__ Unit mine;
  if (wv == 0) {
    const Unit u = unit_by_length(valid_len, p, per_row, blockIdx.x, gridDim.x);
    if ((threadIdx.x & 63) == 0) mine = u;
  }
  __syncthreads();
  return {__builtin_amdgcn_readfirstlane(mine.id), __builtin_amdgcn_readfirstlane(mine.valid)};
}

}  // namespace

// =============================================================================================
// forward
// =============================================================================================
// PERPOS: the long-term branch takes one selection row per query POSITION and key/value group (the
// selection rule as printed, Eq. 8-13 with Eq. 4-5): K and V are [B,G,L,d], `sel` is [B,G,L,k] with
// selection blocks of BK positions; head h reads the keys and values of group h / (H/G).
// `parts` workgroups share the query tiles of a head.  sel == nullptr: dense causal attention.
// RES: the workgroup stages the keys and values in LDS first, and serves all hpg query heads that read them.
// ORDER: see HEADS BY LENGTH (a kernel of its own, as in the backward: beside it, never taken, the code cost selection + forward at B=225 H=8
// d=8 L=200 2 %).
template <typename T, int D, int BK, bool PERPOS, bool RES, bool ORDER>
__global__ __launch_bounds__(64 * kMaxWaves) __attribute__((amdgpu_waves_per_eu(D == 32 ? 5 : 6))) void fwd_small_kernel(
    const T *__restrict__ Q, const T *__restrict__ K, const T *__restrict__ V, const int *__restrict__ valid_len,
    const int *__restrict__ sel, const float *__restrict__ gate_w, const float *__restrict__ gate_b,
    T *__restrict__ O, float *__restrict__ o_lt_out, float *__restrict__ o_st_out, float *__restrict__ lse_lt_out,
    float *__restrict__ lse_st_out, int hpg, int parts, KParams p)
{
  constexpr int CPL = Geo<D>::CPL, NMB = Geo<D>::NMB, NACC = Geo<D>::NACC;
  extern __shared__ __attribute__((aligned(16))) float small_lds[];  // RES: K and V rows; then the wavefronts' selection words
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), W = blockDim.x >> 6;
  // (one workgroup to a head: the map is the identity, at the price of three divisions, some 75 dependent scalar instructions before
  // the first load: selection + forward at B=40 H=8 L=170 d=16 b=8 17.9 us with it, 17.6 without.  With rows of 128 bytes, d = 32 in
  // fp32, it is the other way round: L=87 b=16 15.7 and 16.0.)
  constexpr bool direct = RES && D * sizeof(T) < 128;
  unsigned vid;
  int valid;
  if constexpr (ORDER) {
    const Unit u = place_by_length(valid_len, p, p.H / hpg, wv);
    vid = (unsigned)u.id;
    valid = u.valid;
  } else vid = direct ? blockIdx.x : mfma::xcd_spread(blockIdx.x, gridDim.x / parts, parts);
  if constexpr (direct) parts = 1;
  const int heads = RES ? hpg : 1;  // query heads of this workgroup
  const int bh0 = (int)(vid / parts) * heads, part = (int)(vid % parts);
  const int b = bh0 / p.H;
  const int NT = (p.L + kTile - 1) / kTile;
  if constexpr (!ORDER) valid = clamp_len(valid_len[b], p.L);
  const int p0 = p.L - valid;
  const int T0 = p0 / kTile;  // (beyond the last tile of a row without a valid position)
  const int q = lane & 15, g = lane >> 4;
  const int kvh = PERPOS ? bh0 / hpg : bh0;
  const bool dense = sel == nullptr;
  const int row_lo = (p.NB - p.nq) * BK;  // first row that is written (serving mode: the last block's)
  const T *Kh = K + (size_t)kvh * p.L * D, *Vh = V + (size_t)kvh * p.L * D;
  const int pitch = RES ? NT * kTile * kLdsRow<T, D> : 0;  // floats of a staged tensor
  if constexpr (RES) {
    stage_pair<T, D, false>(Kh, Vh, small_lds, small_lds + pitch, p.L, T0, NT, p0, lane, wv, W);
    __syncthreads();
  }
  using TileRows = std::conditional_t<RES, LdsRows<T, D>, Rows<T, D>>;
  const TileRows Kr = [&] {
    if constexpr (RES) return LdsRows<T, D>(small_lds, q, g);
    else return Rows<T, D>(Kh, p.L, q, g);
  }();
  const TileRows Vr = [&] {
    if constexpr (RES) return LdsRows<T, D>(small_lds + pitch, q, g);
    else return Rows<T, D>(Vh, p.L, q, g);
  }();
  using Ops = Operands<T, D>;
  const float c2 = p.scale * kLog2eF, kc = Ops::kBf ? c2 : 1.0f;  // (kc: what a product of rows is still to be multiplied by)
  const LaneMasks lm = LaneMasks::make(p, q, g);
  unsigned *my_lds = reinterpret_cast<unsigned *>(small_lds + 2 * pitch) + wv * lt_words(p, PERPOS);

  for (int hh = 0; hh < heads; ++hh)
  for (int u = part * W + wv; NT - 1 - u >= row_lo / kTile; u += parts * W) {
    const int bh = bh0 + hh, h = bh % p.H;
    const Slice Qs(Q + (size_t)bh * p.L * D, (size_t)p.L * D * sizeof(T));
    const int I = NT - 1 - u;
    const int iq = I * kTile + q;
    const bool active = iq < p.L && iq >= p0;
    if (I < T0 || p0 >= p.L) {  // no valid query: outputs are zero
      const int r_lo = max(I * kTile, row_lo), rows = min(I * kTile + kTile, p.L) - r_lo;
      const size_t r0 = (size_t)bh * p.L + r_lo;
      const int el = fresh_lane();
      zero_fill(O + r0 * D, rows * D, el);
      if (o_lt_out) zero_fill(o_lt_out + r0 * D, rows * D, el);
      if (o_st_out) zero_fill(o_st_out + r0 * D, rows * D, el);
      if (el < rows) {
        if (lse_lt_out) lse_lt_out[r0 + el] = 0.0f;
        if (lse_st_out) lse_st_out[r0 + el] = 0.0f;
      }
      continue;
    }
    typename Ops::Row qf;
    load_op<T, D>(Qs, active ? (unsigned)(iq * D + CPL * g) * (unsigned)sizeof(T) : kNowhere, qf);
    LtSel<BK, PERPOS> ls;
    if (!dense) {
      if constexpr (PERPOS) {
        int first[LtSel<BK, PERPOS>::kFirst];
        ls.request(p, sel + (size_t)kvh * p.L * p.k, I, iq, lane, first);
        ls.build(p, my_lds, nullptr, sel + ((size_t)kvh * p.L + min(iq, p.L - 1)) * p.k, active, I, iq, p0, lane, first);
      } else {
        ls.build(p, my_lds, sel + ((size_t)bh * p.NB + I * (kTile / BK)) * p.k, I, p0, lane);
      }
    }
    Ops::scale(qf, c2);
    const int kid_q = mask_block(p, iq);
    const int J_hi = p.bidir ? NT - 1 : I;
    // the walk of word w
    Walk wk;
    auto word = [&](int w, bool dia) __attribute__((always_inline)) {
      const int t = w * 64 + lane;
      // (two query blocks per tile: a row's sums must not depend on what the other block selected, which the serving mode does
      // not know, so every short-term tile is general there and the order of the walk follows from the geometry)
      const bool edge = (t == T0) | (t == I) | (t >= min(NT - 1, p.last_lo / kTile));
      wk.start<false, BK < kTile && !PERPOS>(p, I, w, T0, J_hi, lane, dense || ls.has_tile(min(t, NT - 1)), edge, dia, !dense);
    };
    f32x4 a_lt[NACC], a_st[NACC];
    clear(a_lt);
    clear(a_st);
    float l_lt = 0.0f, l_st = 0.0f, ref_lt = 0.0f, ref_st = 0.0f, s_max = 0.0f;
    typename Ops::Row kf;
    typename Ops::Col vf[NMB];
    auto logits = [&]() -> f32x4 { return Ops::dot(kf, qf, f32x4{0.f, 0.f, 0.f, 0.f}); };  // (times kc)
    auto add_lt = [&](const float (&e)[4]) __attribute__((always_inline)) {
      l_lt += (e[0] + e[1]) + (e[2] + e[3]);
      Ops::add(vf, e, a_lt);
    };
    auto add_st = [&](const float (&e)[4]) __attribute__((always_inline)) {
      l_st += (e[0] + e[1]) + (e[2] + e[3]);
      Ops::add(vf, e, a_st);
    };
    // visibility of this lane's four keys of a general tile: element by element, and as bits where distances decide (`near`)
    auto see = [&](int t, bool (&v_lt)[4], bool (&v_st)[4]) __attribute__((always_inline)) {
      const int key0 = t * kTile + 4 * g;
      const unsigned span = (unsigned)((p.bidir ? p.L - 1 : iq) - p0);
      bool s_lt = wk.is_lt(t);
      if ((PERPOS || BK < kTile) && !dense) s_lt &= ls.sees(q, key0);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const bool ok = (unsigned)(key0 + r - p0) <= span;
        v_lt[r] = ok & s_lt;
        v_st[r] = ok & st_sees(p, iq, key0 + r, kid_q, mask_block(p, key0, r), key0 + r >= p.last_lo);
      }
    };
    auto see_near = [&](int t, unsigned &v_lt, unsigned &v_st) __attribute__((always_inline)) {
      const int key0 = t * kTile + 4 * g;
      const unsigned ok = LaneMasks::keys(p, key0, p0, iq);
      v_st = (lm.st(p, I - t) | LaneMasks::from(p.last_lo - key0)) & ok;
      bool s_lt = wk.is_lt(t);
      if ((PERPOS || BK < kTile) && !dense) s_lt &= ls.sees(q, key0);
      v_lt = s_lt ? ok : 0u;
    };
    // one tile: the next one's keys are requested as soon as this one's are in the matrix cores, its values at the end
    auto body = [&](auto kind, auto unit, Word &mask) __attribute__((always_inline)) {
      constexpr int KIND = decltype(kind)::value;
      constexpr bool UNIT = decltype(unit)::value;
      const int t = wk.take(mask), t_next = wk.peek();
      const f32x4 s = logits();
      Kr.op(t_next, kf);
      if constexpr (TileRows::kNear) Vr.col(t, vf);
      s_max = fmaxf(fmaxf(s_max, fabsf(s[0])), fabsf(s[1]));
      s_max = fmaxf(fmaxf(s_max, fabsf(s[2])), fabsf(s[3]));
      float e[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) e[r] = __builtin_amdgcn_exp2f(kc * s[r]);
      if constexpr (KIND == 0) {
        float el[4], es[4];
        if constexpr (UNIT) {
          unsigned v_lt, v_st;
          see_near(t, v_lt, v_st);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            el[r] = keep(e[r], v_lt, r);
            es[r] = keep(e[r], v_st, r);
          }
        } else {
          bool v_lt[4], v_st[4];
          see(t, v_lt, v_st);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            el[r] = v_lt[r] ? e[r] : 0.0f;
            es[r] = v_st[r] ? e[r] : 0.0f;
          }
        }
        add_lt(el);
        add_st(es);
      } else if constexpr (KIND == 1) {
        if constexpr (PERPOS || BK < kTile) {
          const bool v = dense || ls.sees(q, t * kTile + 4 * g);
#pragma unroll
          for (int r = 0; r < 4; ++r) e[r] = v ? e[r] : 0.0f;
        }
        add_lt(e);
      } else {
        if constexpr (UNIT) {
          const unsigned v = lm.st(p, I - t);
#pragma unroll
          for (int r = 0; r < 4; ++r) e[r] = keep(e[r], v, r);
        } else {
          const int key0 = t * kTile + 4 * g;
#pragma unroll
          for (int r = 0; r < 4; ++r) e[r] = st_sees(p, iq, key0 + r, kid_q, mask_block(p, key0, r), false) ? e[r] : 0.0f;
        }
        add_st(e);
      }
      if constexpr (!TileRows::kNear) Vr.col(t_next, vf);
    };
    auto walk = [&](auto unit) __attribute__((always_inline)) {
      for (int w = T0 >> 6; w <= J_hi >> 6; ++w) {
        word(w, false);
        if (!wk.all()) continue;
        const int t = wk.peek();
        Kr.op(t, kf);
        if constexpr (!TileRows::kNear) Vr.col(t, vf);
        while (wk.m0) body(std::integral_constant<int, 0>{}, unit, wk.m0);
        while (wk.m1) body(std::integral_constant<int, 1>{}, unit, wk.m1);
        while (wk.m2) body(std::integral_constant<int, 2>{}, unit, wk.m2);
      }
    };
    auto far_keys = [&]() __attribute__((always_inline)) {
      float qd[CPL];
      Ops::floats(qf, qd);
      float qw[CPL * 4];
      if constexpr (D == 8) whole_row(qd, qw);
      diagonals(p, I, T0, J_hi, [&](int d) __attribute__((always_inline)) {
        if constexpr (D == 8) {
          const int t = min(max(I + d * (1 << g), T0), NT - 1), key = iq + kTile * d * (1 << g);
          float kr[D], vr[D];
          Kr.whole(t, kr);
          Vr.whole(t, vr);
          const float x = dot_n(qw, kr, 0.0f);
          const bool ok = active & (key >= p0) & (key < p.last_lo);
          s_max = fmaxf(s_max, ok ? fabsf(x) : 0.0f);
          const float ex = ok ? __builtin_amdgcn_exp2f(kc * x) : 0.0f;
          l_st += ex;
          add_row(a_st, ex, vr);
          return;
        } else {
        float s[4], e[4], vo[4][NMB][4];
#pragma unroll
        for (int n = 0; n < 4; ++n) {
          float kr[CPL];
          Kr.row(min(max(I + d * (1 << n), T0), NT - 1), kr);
          s[n] = dot_n(qd, kr, 0.0f);
        }
        phase_end<D>();
#pragma unroll
        for (int n = 0; n < 4; ++n) Vr.own(min(max(I + d * (1 << n), T0), NT - 1), vo[n]);
        const float x = gather_g(s);
        const int key = iq + kTile * d * (1 << g);
        const bool ok = active & (key >= p0) & (key < p.last_lo);
        s_max = fmaxf(s_max, ok ? fabsf(x) : 0.0f);
        const float ex = ok ? __builtin_amdgcn_exp2f(kc * x) : 0.0f;
        l_st += ex;
        spread_g(ex, e);
        add_own(a_st, e, vo);
        }
      });
    };
    constexpr bool far_first = D == 32 && Ops::kBf;
    if (far_first && p.sblk == 1 && !dense) far_keys();
    if (p.sblk <= 1) walk(std::true_type{});
    else walk(std::false_type{});
    if (!far_first && p.sblk == 1 && !dense) far_keys();
    if (__builtin_expect(!__all(s_max * kc <= kSmallLogit && abs_sum(a_lt) + abs_sum(a_st) < 1.0e37f), 0)) {
      // large logits, or values near the end of fp32's range or beyond: the row maxima of both branches, then the walk
      // against them
      float x_lt = kNegInfF, x_st = kNegInfF;
      auto each = [&](auto f) __attribute__((always_inline)) {
        for (int w = T0 >> 6; w <= J_hi >> 6; ++w) {
          word(w, true);
          for (Word m = wk.all(); m;) f(wk.take(m));
        }
      };
      each([&](int J) {
        Kr.op(J, kf);
        const f32x4 s = logits() * kc;
        bool v_lt[4], v_st[4];
        see(J, v_lt, v_st);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          x_lt = fmaxf(x_lt, v_lt[r] ? s[r] : kNegInfF);
          x_st = fmaxf(x_st, v_st[r] ? s[r] : kNegInfF);
        }
      });
      x_lt = max_g(x_lt);
      x_st = max_g(x_st);
      ref_lt = x_lt == kNegInfF ? 0.0f : x_lt;
      ref_st = x_st == kNegInfF ? 0.0f : x_st;
      l_lt = l_st = 0.0f;
      clear(a_lt);
      clear(a_st);
      each([&](int J) {
        Kr.op(J, kf);
        Vr.col(J, vf);
        const f32x4 s = logits() * kc;
        float lost[4];
        take_out<T, D>(vf, g, lost);
        bool v_lt[4], v_st[4];
        see(J, v_lt, v_st);
        float el[4], es[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          el[r] = v_lt[r] ? __builtin_amdgcn_exp2f(s[r] - ref_lt) + lost[r] : 0.0f;
          es[r] = v_st[r] ? __builtin_amdgcn_exp2f(s[r] - ref_st) + lost[r] : 0.0f;
        }
        add_lt(el);
        add_st(es);
      });
#pragma unroll
      for (int mb = 0; mb < NACC; ++mb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {  // (a row of the padding may have seen some of the padding)
          a_lt[mb][r] = active ? a_lt[mb][r] : 0.0f;
          a_st[mb][r] = active ? a_st[mb][r] : 0.0f;
        }
    }
    // closes a branch: normalised output, returns the row's sum (both zero for rows that take no part)
    f32x4 o_lt[NMB], o_st[NMB];
    auto finish = [&](const f32x4 (&part)[NACC], f32x4 (&acc)[NMB], float l) -> float {
      total<D>(part, acc);
      const float lt = sum_g(l);
      const bool ok = active && !(lt <= 0.0f);  // (a NaN stays one)
      const float inv = ok ? recip(lt) : 0.0f;
#pragma unroll
      for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[mb][r] *= inv;
      return ok ? lt : 0.0f;
    };
    // log sum exp from a row's sum.  The hardware's logarithm is off by an ulp of its own size, some 5, and every probability of the
    // backward would carry that: what it misses is l * 2^-log - 1 (errors against 64 bits 0.6 of those without, of dQ, dK and dV 0.9;
    // 0.05 us of a call of 6).
    auto lse = [&](float l, float m) -> float {
      const float log = __builtin_amdgcn_logf(l), missed = fmaf(l, __builtin_amdgcn_exp2f(-log), -1.0f);
      return l == 0.0f ? 0.0f : fmaf(m + log, kLn2F, fmaf(m + log, kLn2Low, missed));
    };
    const int el = fresh_lane(), eg = el >> 4, ei = I * kTile + (el & 15);
    const bool in_range = ei < p.L && ei >= row_lo;
    const size_t lrow = (size_t)bh * p.L + ei, rowoff = lrow * D;
    const float sum_lt = finish(a_lt, o_lt, l_lt);
    if (dense) {
      if (in_range) store_row4<T, D>(O + rowoff, o_lt, eg);
      if (in_range && eg == 0 && lse_lt_out) lse_lt_out[lrow] = lse(sum_lt, ref_lt);
      continue;
    }
    const float sum_st = finish(a_st, o_st, l_st);

    // ---- gate and blend (Eq. 18-19) ----
    const float *wl = gate_w + (size_t)h * 2 * D;
    float z = 0.0f;
#pragma unroll
    for (int mb = 0; mb < NMB; ++mb)
      if (16 * mb + 4 * eg < D) {
        float x[4], y[4];
        load_n<4>(wl + 16 * mb + 4 * eg, x);
        load_n<4>(wl + D + 16 * mb + 4 * eg, y);
#pragma unroll
        for (int r = 0; r < 4; ++r) z = fmaf(y[r], o_st[mb][r], fmaf(x[r], o_lt[mb][r], z));
      }
    z = sum_g(z) + (gate_b ? gate_b[h] : 0.0f);
    const float alpha = sigmoid(z);
    if (in_range) {
      if (o_lt_out) store_row4<float, D, true>(o_lt_out + rowoff, o_lt, eg);
      if (o_st_out) store_row4<float, D, true>(o_st_out + rowoff, o_st, eg);
      f32x4 o[NMB];
#pragma unroll
      for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
        for (int r = 0; r < 4; ++r) o[mb][r] = alpha * o_lt[mb][r] + (1.0f - alpha) * o_st[mb][r];
      store_row4<T, D>(O + rowoff, o, eg);
      if (eg == 0) {
        if (lse_lt_out) lse_lt_out[lrow] = lse(sum_lt, ref_lt);
        if (lse_st_out) lse_st_out[lrow] = lse(sum_st, ref_st);
      }
    }
  }
}

// =============================================================================================
// forward, THE NEAR FORM (see there)
// =============================================================================================
// A query tile walks the tile before, itself, its long-term tiles below (the first valid one, which may hold padding, first) and the
// diagonals.  (The tile before first: its terms are the smaller ones, and what is added after a large sum is rounded at that sum's size.  The
// other way round o_st of bf16 at d = 32 under mask block 1 errs 1.03 times as much.)
// Bound by the latency of a wavefront's own chain at three to four wavefronts a SIMD (half of their time went on waits, 566 vector and
// 420 scalar instructions a tile) rather than by a pipe, so:
//  - What a tile needs from memory is requested a tile ahead and has arrived before the stores go out: loads and stores finish in
//    order, and a wait for loads issued behind a tile's stores was a wait for those stores.
//  - The selection is read from registers, entry by entry, where LDS words were cleared, set by atomics and read back.
//  - Masks are scalars, the walk is three straight pieces, row sums and the lse of both branches are closed together.
// us, with fwd_small_kernel / with this: B=256 H=2 L=200 d=32 19.5 / 18.1, B=2048 H=8 L=200 d=16 283 / 219, per position at d=8 238 /
// 194, B=32 H=8 L=2000 d=8 (streamed) 58.8 / 52.9; selection + forward at B=4 H=2 L=50 d=32 10.1 / 9.3.
template <typename T, int D, int BK, bool PERPOS, bool RES, bool ORDER>
__global__ __launch_bounds__(64 * kMaxWaves) __attribute__((amdgpu_waves_per_eu(D == 32 || (RES && PERPOS) ? 4 : 5))) void fwd_near_kernel(
    const T *__restrict__ Q, const T *__restrict__ K, const T *__restrict__ V, const int *__restrict__ valid_len,
    const int *__restrict__ sel, const float *__restrict__ gate_w, const float *__restrict__ gate_b,
    T *__restrict__ O, float *__restrict__ o_lt_out, float *__restrict__ o_st_out, float *__restrict__ lse_lt_out,
    float *__restrict__ lse_st_out, int hpg, int parts, NearMasks nm, KParams p)
{
  constexpr int CPL = Geo<D>::CPL, NMB = Geo<D>::NMB, NACC = Geo<D>::NACC;
  constexpr bool kPicked = !PERPOS && BK == kTile;
  using Ops = Operands<T, D>;
  using Sel = LtSel<BK, PERPOS>;
  extern __shared__ __attribute__((aligned(16))) float small_lds[];  // RES: K and V rows; then the wavefronts' selection words
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), W = blockDim.x >> 6;
  constexpr bool direct = RES && D * sizeof(T) < 128;  // (see fwd_small_kernel)
  unsigned vid;
  int valid;
  if constexpr (ORDER) {
    const Unit u = place_by_length(valid_len, p, p.H / hpg, wv);
    vid = (unsigned)u.id;
    valid = u.valid;
  } else vid = direct ? blockIdx.x : mfma::xcd_spread(blockIdx.x, gridDim.x / parts, parts);
  if constexpr (RES) parts = 1;
  const int heads = RES && PERPOS ? hpg : 1;  // query heads of this workgroup
  const int bh0 = (int)(vid / parts) * heads, part = (int)(vid % parts);
  const int NT = (p.L + kTile - 1) / kTile;
  if constexpr (!ORDER) valid = clamp_len(valid_len[bh0 / p.H], p.L);
  const int p0 = p.L - valid;
  const int T0 = p0 / kTile;  // (beyond the last tile of a row without a valid position)
  const int q = lane & 15, g = lane >> 4;
  const int kvh = PERPOS ? bh0 / hpg : bh0;
  const int row_lo = (p.NB - p.nq) * BK;  // first row that is written (serving mode: the last block's)
  const int I_lo = row_lo / kTile;
  const T *Kh = K + (size_t)kvh * p.L * D, *Vh = V + (size_t)kvh * p.L * D;
  const int pitch = RES ? NT * kTile * kLdsRow<T, D> : 0;  // floats of a staged tensor

  // what a query tile needs from memory, requested a tile ahead
  struct Request {
    typename Ops::Row q;
    int sel[Sel::kFirst];
    __device__ __forceinline__ void arrived()
    {
      Ops::arrived(q);
      arrive(sel);
    }
  };
  const int *sel_unit = sel + (PERPOS ? (size_t)kvh * p.L : (size_t)bh0 * p.NB) * p.k;
  auto request = [&](int hh, int I, Request &x) __attribute__((always_inline)) {  // (any I: see QueryIn)
    const int iq = I * kTile + q;
    const Slice Qs(Q + (size_t)(bh0 + hh) * p.L * D, (size_t)p.L * D * sizeof(T));
    load_op<T, D>(Qs, iq < p.L && iq >= p0 ? (unsigned)(iq * D + CPL * g) * (unsigned)sizeof(T) : kNowhere, x.q);
    Sel::request(p, sel_unit, max(I, 0), max(iq, 0), lane, x.sel);
    asm volatile("" ::: "memory");
  };
  // the (tile, head) pairs of the workgroup in turn, its wavefronts one each; the next one of this wavefront's
  struct Item {
    int I, hh;
  };
  const int dI = parts * W / heads, dh = parts * W - dI * heads;
  auto item_after = [&](Item x) -> Item {
    if (heads == 1) return {x.I - dI, 0};
    x.hh += dh;
    return x.hh >= heads ? Item{x.I - dI - 1, x.hh - heads} : Item{x.I - dI, x.hh};
  };
  const int start = part * W + wv;
  Item it{NT - 1 - start / heads, start % heads};
  Request now;
  request(it.hh, it.I, now);
  if constexpr (RES) {
    stage_pair<T, D, false, kStageAhead<D>>(Kh, Vh, small_lds, small_lds + pitch, p.L, T0, NT, p0, lane, wv, W);
    __syncthreads();
  }
  using TileRows = std::conditional_t<RES, LdsRows<T, D>, Rows<T, D>>;
  const TileRows Kr = [&] {
    if constexpr (RES) return LdsRows<T, D>(small_lds, q, g);
    else return Rows<T, D>(Kh, p.L, q, g);
  }();
  const TileRows Vr = [&] {
    if constexpr (RES) return LdsRows<T, D>(small_lds + pitch, q, g);
    else return Rows<T, D>(Vh, p.L, q, g);
  }();
  const float c2 = p.scale * kLog2eF, kc = Ops::kBf ? c2 : 1.0f;  // (kc: what a product of rows is still to be multiplied by)
  unsigned *my_lds = reinterpret_cast<unsigned *>(small_lds + 2 * pitch) + wv * lt_words(p, PERPOS);
  Word valid_keys[4];  // of the first tile
#pragma unroll
  for (int r = 0; r < 4; ++r) valid_keys[r] = elements_from(p0 & (kTile - 1), r);

  const int I_first = p0 >= p.L ? NT : max(I_lo, T0);
  const int h0 = bh0 % p.H;
  for (; it.I >= I_first; it = item_after(it)) {
    const int I = it.I, hh = it.hh, bh = bh0 + hh;
    const int iq = I * kTile + q;
    const bool active = iq < p.L && iq >= p0;
    typename Ops::Row qf = now.q;
    int first[Sel::kFirst];
#pragma unroll
    for (int i = 0; i < Sel::kFirst; ++i) first[i] = now.sel[i];
    const Item next = item_after(it);
    request(next.hh, next.I, now);
    Sel ls;
    if constexpr (!kPicked)
      ls.build(p, my_lds, PERPOS ? nullptr : sel_unit + (size_t)I * (kTile / BK) * p.k, sel_unit + (size_t)min(iq, p.L - 1) * p.k, active, I, iq,
               p0, lane, first);
    // the head's gate
    const int h = h0 + hh;
    const float *wg = gate_w + (size_t)h * 2 * D + (4 * g & (D - 1));
    const float bias = gate_b ? gate_b[h] : 0.0f;
    float w_lt[NMB][4], w_st[NMB][4];
#pragma unroll
    for (int mb = 0; mb < NMB; ++mb) {
      load_n<4>(wg + 16 * mb, w_lt[mb]);
      load_n<4>(wg + 16 * mb + D, w_st[mb]);
    }
    asm volatile("" ::: "memory");
    Ops::scale(qf, c2);
    // the long-term tiles of word w, whatever else the entries name
    auto tiles_of = [&](int w) __attribute__((always_inline)) -> Word {
      if constexpr (kPicked) return PickedTiles{sel_unit + (size_t)I * p.k, p.k, first[0]}.word(w, lane);
      else if constexpr (PERPOS) return ls.all;
      else return __ballot(ls.has_tile(min(w * 64 + lane, NT - 1)));
    };
    f32x4 a_lt[NACC], a_st[NACC];
    clear(a_lt);
    clear(a_st);
    float l_lt = 0.0f, l_st = 0.0f, ref_lt = 0.0f, ref_st = 0.0f, s_max = 0.0f;
    typename Ops::Row kf;
    typename Ops::Col vf[NMB];
    auto logits = [&]() -> f32x4 { return Ops::dot(kf, qf, f32x4{0.f, 0.f, 0.f, 0.f}); };  // (times kc)
    auto add_lt = [&](const float (&e)[4]) __attribute__((always_inline)) {
      l_lt += (e[0] + e[1]) + (e[2] + e[3]);
      Ops::add(vf, e, a_lt);
    };
    auto add_st = [&](const float (&e)[4]) __attribute__((always_inline)) {
      l_st += (e[0] + e[1]) + (e[2] + e[3]);
      Ops::add(vf, e, a_st);
    };
    // one tile; the next one's keys are requested as soon as this one's are in the matrix cores, its values at the end
    auto tile = [&](auto lt, auto st, auto masked, int t, int t_next, const Word (&m_lt)[4], const Word (&m_st)[4])
                    __attribute__((always_inline)) {
      constexpr bool LT = decltype(lt)::value, ST = decltype(st)::value, MASKED = decltype(masked)::value;
      const f32x4 s = logits();
      Kr.op(t_next, kf);
      if constexpr (TileRows::kNear) Vr.col(t, vf);
      // (the request is not moved down to that of the next values, where the compiler has it at d = 16: lists of 61 at L=2114, the last block
      // alone, 20.3 us with and 17.5 without that)
      else if constexpr (D == 16) asm volatile("" ::: "memory");
      s_max = fmaxf(fmaxf(s_max, fabsf(s[0])), fabsf(s[1]));
      s_max = fmaxf(fmaxf(s_max, fabsf(s[2])), fabsf(s[3]));
      float e[4], el[4], es[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) e[r] = __builtin_amdgcn_exp2f(kc * s[r]);
      bool mine = true;
      if constexpr (LT && (PERPOS || BK < kTile)) mine = ls.sees(q, t * kTile + 4 * g);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if constexpr (LT) el[r] = mine && (!MASKED || in_lanes(m_lt[r])) ? e[r] : 0.0f;
        if constexpr (ST) es[r] = in_lanes(m_st[r]) ? e[r] : 0.0f;
      }
      if constexpr (LT) add_lt(el);
      if constexpr (ST) add_st(es);
      if constexpr (!TileRows::kNear) Vr.col(t_next, vf);
    };
    auto walk = [&]() __attribute__((always_inline)) {
      constexpr auto yes = std::true_type{};
      constexpr auto no = std::false_type{};
      constexpr bool kOneWord = RES || PERPOS;
      const int w0 = kOneWord ? 0 : T0 >> 6, wI = kOneWord ? 0 : I >> 6;
      Kr.op(max(I - 1, T0), kf);
      if constexpr (!TileRows::kNear) Vr.col(max(I - 1, T0), vf);
      const Word at_I = tiles_of(wI);
      const bool own = (at_I >> (I & 63)) & 1ull;
      const bool before = (wI != w0 && (I & 63) == 0 ? tiles_of(wI - 1) : at_I) >> ((I - 1) & 63) & 1ull;
      // of word w, the tiles from the first valid one to the last but one before I
      auto rest_of = [&](int w) __attribute__((always_inline)) -> Word {
        Word m = w == wI ? at_I : tiles_of(w);
        if (w == w0) m &= ~0ull << (T0 & 63);
        if (w == (I - 1) >> 6) m &= (1ull << ((I - 1) & 63)) - 1ull;
        return w > (I - 1) >> 6 ? 0ull : m;
      };
      Word rest = I > T0 ? rest_of(w0) : 0ull;
      auto next_of = [&](int w, Word m) __attribute__((always_inline)) -> int { return m ? 64 * w + __builtin_ctzll(m) : I; };
      Word m_lt[4], m_st[4];
      if (I > T0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          m_lt[r] = I - 1 == T0 ? valid_keys[r] : ~0ull;
          m_st[r] = nm.next[r] & m_lt[r];
        }
        if (before) tile(yes, yes, yes, I - 1, I, m_lt, m_st);
        else tile(no, yes, yes, I - 1, I, m_lt, m_st);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const Word ok = I == T0 ? valid_keys[r] : ~0ull;
        m_lt[r] = own ? triangle(r, false) & ok : 0ull;
        m_st[r] = nm.own[r] & ok;
      }
      tile(yes, yes, yes, I, next_of(w0, rest), m_lt, m_st);
      if (I == T0) return;
      for (int w = w0;;) {
        if (w == w0 && (rest >> (T0 & 63)) & 1ull) {
          rest &= rest - 1;
          tile(yes, no, yes, T0, next_of(w, rest), valid_keys, valid_keys);
        }
        while (rest) {
          const int t = 64 * w + __builtin_ctzll(rest);
          rest &= rest - 1;
          tile(yes, no, no, t, next_of(w, rest), m_lt, m_st);
        }
        if (kOneWord || ++w > wI) break;
        rest = rest_of(w);
        Kr.op(next_of(w, rest), kf);
        if constexpr (!TileRows::kNear) Vr.col(next_of(w, rest), vf);
      }
    };
    auto far_keys = [&]() __attribute__((always_inline)) {
      float qd[CPL];
      Ops::floats(qf, qd);
      float qw[CPL * 4];
      if constexpr (D == 8) whole_row(qd, qw);
      diagonals(p, I, T0, I, [&](int d) __attribute__((always_inline)) {
        const int key = iq + kTile * d * (1 << g);
        const bool ok = active & (key >= p0);
        if constexpr (D == 8) {
          const int t = max(I + d * (1 << g), T0);
          float kr[D], vr[D];
          Kr.whole(t, kr);
          Vr.whole(t, vr);
          const float x = dot_n(qw, kr, 0.0f);
          s_max = fmaxf(s_max, ok ? fabsf(x) : 0.0f);
          const float ex = ok ? __builtin_amdgcn_exp2f(kc * x) : 0.0f;
          l_st += ex;
          add_row(a_st, ex, vr);
        } else {
          float s[4], e[4], vo[4][NMB][4];
#pragma unroll
          for (int n = 0; n < 4; ++n) {
            float kr[CPL];
            Kr.row(max(I + d * (1 << n), T0), kr);
            s[n] = dot_n(qd, kr, 0.0f);
          }
          phase_end<D>();
#pragma unroll
          for (int n = 0; n < 4; ++n) Vr.own(max(I + d * (1 << n), T0), vo[n]);
          const float x = gather_g(s);
          s_max = fmaxf(s_max, ok ? fabsf(x) : 0.0f);
          const float ex = ok ? __builtin_amdgcn_exp2f(kc * x) : 0.0f;
          l_st += ex;
          spread_g(ex, e);
          add_own(a_st, e, vo);
        }
      });
    };
    constexpr bool far_first = D == 32 && Ops::kBf;
    if (far_first && p.sblk == 1) far_keys();
    walk();
    if (!far_first && p.sblk == 1) far_keys();
    if (__builtin_expect(__ballot(!((s_max * kc <= kSmallLogit) & (abs_sum(a_lt) + abs_sum(a_st) < 1.0e37f))) != 0ull, 0)) {
      // large logits, or values near the end of fp32's range or beyond: the row maxima of both branches, then the walk
      // against them, tile by tile with every test
      float x_lt = kNegInfF, x_st = kNegInfF;
      auto each = [&](auto f) __attribute__((always_inline)) {
        for (int w = T0 >> 6; w <= I >> 6; ++w) {
          const Word lt = tiles_of(w);
          // the tiles of either branch, from T0 to I: of the short-term one those at distances 0 and 1 and, with all of Eq. 15, 2^r
          Word m = lt;
          for (int d = 0; I - d >= T0; d = d ? 2 * d : 1) {
            if ((I - d) >> 6 == w) m |= 1ull << ((I - d) & 63);
            if (d == 1 && p.sblk != 1) break;
          }
          if (w == T0 >> 6) m &= ~0ull << (T0 & 63);
          if (w == I >> 6) m &= ~0ull >> (63 - (I & 63));
          for (; m; m &= m - 1) {
            const int t = 64 * w + __builtin_ctzll(m);
            const bool in_lt = (lt >> (t & 63)) & 1ull;
            Kr.op(t, kf);
            const f32x4 s = logits() * kc;
            const int key0 = t * kTile + 4 * g;
            bool s_lt = in_lt, v_lt[4], v_st[4];
            if (PERPOS || BK < kTile) s_lt &= ls.sees(q, key0);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int dist = iq - (key0 + r);
              const bool ok = (dist >= 0) & (key0 + r >= p0);
              v_lt[r] = ok & s_lt;
              v_st[r] = ok & ((dist < p.w) | ((p.sblk == 1) & (__popc(dist) == 1)));
            }
            f(t, s, v_lt, v_st);
          }
        }
      };
      each([&](int, const f32x4 &s, const bool (&v_lt)[4], const bool (&v_st)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          x_lt = fmaxf(x_lt, v_lt[r] ? s[r] : kNegInfF);
          x_st = fmaxf(x_st, v_st[r] ? s[r] : kNegInfF);
        }
      });
      x_lt = max_g(x_lt);
      x_st = max_g(x_st);
      ref_lt = x_lt == kNegInfF ? 0.0f : x_lt;
      ref_st = x_st == kNegInfF ? 0.0f : x_st;
      l_lt = l_st = 0.0f;
      clear(a_lt);
      clear(a_st);
      each([&](int t, const f32x4 &s, const bool (&v_lt)[4], const bool (&v_st)[4]) __attribute__((always_inline)) {
        Vr.col(t, vf);
        float lost[4];
        take_out<T, D>(vf, g, lost);
        float el[4], es[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          el[r] = v_lt[r] ? __builtin_amdgcn_exp2f(s[r] - ref_lt) + lost[r] : 0.0f;
          es[r] = v_st[r] ? __builtin_amdgcn_exp2f(s[r] - ref_st) + lost[r] : 0.0f;
        }
        add_lt(el);
        add_st(es);
      });
#pragma unroll
      for (int mb = 0; mb < NACC; ++mb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {  // (a row of the padding may have seen some of the padding)
          a_lt[mb][r] = active ? a_lt[mb][r] : 0.0f;
          a_st[mb][r] = active ? a_st[mb][r] : 0.0f;
        }
    }
    // ---- both branches' row sums, long-term in the even lane groups, short-term in the odd ones; the lse and 1 / sum of each ----
    const int el = fresh_lane(), eg = el >> 4, er = el & 15, ei = I * kTile + er;
    float sum;
    {
      const u32x2_t a = __builtin_amdgcn_permlane16_swap(__float_as_uint(l_lt), __float_as_uint(l_st), false, false);
      const unsigned u = __float_as_uint(__uint_as_float(a[0]) + __uint_as_float(a[1]));
      const u32x2_t b = __builtin_amdgcn_permlane32_swap(u, u, false, false);
      sum = __uint_as_float(b[0]) + __uint_as_float(b[1]);
    }
    const bool ok = (ei < p.L) & (ei >= p0) & !(sum <= 0.0f);  // (a NaN stays one)
    const unsigned inv = __float_as_uint(ok ? recip(sum) : 0.0f);
    const u32x2_t invs = __builtin_amdgcn_permlane16_swap(inv, inv, false, false);
    f32x4 o_lt[NMB], o_st[NMB];
    total<D>(a_lt, o_lt);
    total<D>(a_st, o_st);
#pragma unroll
    for (int mb = 0; mb < NMB; ++mb) {
      o_lt[mb] *= __uint_as_float(invs[0]);
      o_st[mb] *= __uint_as_float(invs[1]);
    }

    // ---- gate and blend (Eq. 18-19) ----
    float z = 0.0f;
#pragma unroll
    for (int mb = 0; mb < NMB; ++mb)
      if (16 * mb + 4 * eg < D) {
#pragma unroll
        for (int r = 0; r < 4; ++r) z = fmaf(w_st[mb][r], o_st[mb][r], fmaf(w_lt[mb][r], o_lt[mb][r], z));
      }
    z = sum_g(z) + bias;
    const float alpha = sigmoid(z);
    // (the next tile's rows have arrived before the stores go out: a wait for them behind those would be one for the stores)
    now.arrived();
    if (ei < p.L && ei >= row_lo) {
      const unsigned at = (unsigned)ei * D;
      const size_t head = (size_t)bh * p.L;
      if (o_lt_out) store_row4<float, D, true>(o_lt_out + head * D + at, o_lt, eg);
      if (o_st_out) store_row4<float, D, true>(o_st_out + head * D + at, o_st, eg);
      f32x4 o[NMB];
#pragma unroll
      for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
        for (int r = 0; r < 4; ++r) o[mb][r] = alpha * o_lt[mb][r] + (1.0f - alpha) * o_st[mb][r];
      store_row4<T, D>(O + head * D + at, o, eg);
      // log sum exp from a row's sum (see fwd_small_kernel)
      const float ref = eg == 0 ? ref_lt : ref_st;
      const float log = __builtin_amdgcn_logf(sum), missed = fmaf(sum, __builtin_amdgcn_exp2f(-log), -1.0f);
      const float lse = ok ? fmaf(ref + log, kLn2F, fmaf(ref + log, kLn2Low, missed)) : 0.0f;
      if (lse_lt_out && eg == 0) lse_lt_out[head + (unsigned)ei] = lse;
      if (lse_st_out && eg == 1) lse_st_out[head + (unsigned)ei] = lse;
    }
  }
  // positions before the first tile with a valid one: zeros
  const int end = p0 >= p.L ? p.L : T0 * kTile;
  if (end > row_lo)
    for (int hh = 0; hh < heads; ++hh) {
      const size_t first = (size_t)(bh0 + hh) * p.L + row_lo;
      const int rows = end - row_lo, from = (part * W + wv) * 64 + lane, step = parts * W * 64;
      zero_rows_from(O + first * D, rows * D, from, step);
      if (o_lt_out) zero_rows_from(o_lt_out + first * D, rows * D, from, step);
      if (o_st_out) zero_rows_from(o_st_out + first * D, rows * D, from, step);
      for (int i = from; i < rows; i += step) {
        if (lse_lt_out) lse_lt_out[first + i] = 0.0f;
        if (lse_st_out) lse_st_out[first + i] = 0.0f;
      }
    }
}

// =============================================================================================
// backward of one query tile (gate pass, dQ) and of one key tile (dK, dV)
// =============================================================================================
namespace {

// LDS of bwd_res_kernel, in floats: K and V, per head Q and dO (overlay: in the place of K and V), row constants, tile words and
// selection bits, the wavefronts' selection words
struct ResLayout {
  int pitch, qg, rowc, words, waves, held, gates, red, total;
  // row: floats of a staged row
  __host__ __device__ ResLayout(const KParams &p, int row, bool perpos, int hpg, int overlay, int W)
  {
    const int NT = (p.L + kTile - 1) / kTile, rows = NT * kTile;
    pitch = rows * row;
    qg = overlay ? 0 : 2 * pitch;
    rowc = overlay ? 2 * hpg * pitch : 2 * pitch + 2 * hpg * pitch;
    words = rowc + hpg * 6 * rows;
    waves = words + NT * ((NT + 31) / 32) + (perpos ? 2 * rows : p.b < kTile ? 2 * NT * ((p.NB + 31) / 32) : 0);
    waves = (waves + 3) / 4 * 4;
    held = waves + W * lt_words(p, perpos);
    // (the near form: the heads' gate rows, and every wavefront's gate sums of every head)
    gates = (held + 3) / 4 * 4;
    red = gates + hpg * 2 * p.d;
    total = near_form(p) ? red + hpg * W * (2 * p.d + 1) : held;
  }
};

// one query head as the gate pass and dQ read it
struct QueryHead {
  Slice Q, dO, o_lt, o_st, lse_lt, lse_st;
  template <typename T>
  __device__ __forceinline__ QueryHead(const T *q, const T *g, const float *ol, const float *os, const float *ll, const float *lst, int bh,
                                       int L, int D)
      : Q(q + (size_t)bh * L * D, (size_t)L * D * sizeof(T)), dO(g + (size_t)bh * L * D, (size_t)L * D * sizeof(T)),
        o_lt(ol + (size_t)bh * L * D, (size_t)L * D * 4), o_st(os + (size_t)bh * L * D, (size_t)L * D * 4),
        lse_lt(ll + (size_t)bh * L, (size_t)L * 4), lse_st(lst + (size_t)bh * L, (size_t)L * 4)
  {
  }
};
// the gate of one head, and the running gradient sums of the rows this wavefront took over this lane's channels
template <int D>
struct GateSums {
  const float *w;
  float bias, gl[Geo<D>::CPL], gs[Geo<D>::CPL], gb;
  __device__ __forceinline__ GateSums(const float *gate_w, const float *gate_b, int h) : w(gate_w + (size_t)h * 2 * D)
  {
    bias = gate_b ? gate_b[h] : 0.0f;
    zero_n(gl);
    zero_n(gs);
    gb = 0.0f;
  }
  // this lane's weights, read anew for every tile: in registers through the walk of d = 32 they make others spill
  __device__ __forceinline__ void weights(int g, float (&wl)[Geo<D>::CPL], float (&ws)[Geo<D>::CPL]) const
  {
    int at = Geo<D>::CPL * g;
    asm volatile("" : "+v"(at));
    load_n<Geo<D>::CPL>(w + at, wl);
    load_n<Geo<D>::CPL>(w + at + D, ws);
  }
  // sums over the 16 rows of the lanes, then over the workgroup's W wavefronts in order, to out[2D+1]; red: [kMaxWaves][2D+1] in LDS
  __device__ __forceinline__ void finish(float (*red)[2 * D + 1], float *out, int lane, int wv, int W)
  {
    constexpr int CPL = Geo<D>::CPL, GW = 2 * D + 1;
    const int q = lane & 15, g = lane >> 4;
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
      gl[i] = sum_row(gl[i]);
      gs[i] = sum_row(gs[i]);
    }
    gb = sum_row(gb);
    if (q == 0) {
#pragma unroll
      for (int i = 0; i < CPL; ++i) {
        red[wv][CPL * g + i] = gl[i];
        red[wv][D + CPL * g + i] = gs[i];
      }
      if (g == 0) red[wv][2 * D] = gb;
    }
    __syncthreads();
    for (int c = threadIdx.x; c < GW; c += blockDim.x) {
      float a = 0.0f;
      for (int w = 0; w < W; ++w) a += red[w][c];
      out[c] = a;
    }
  }
};

// Query tile I.  sel_head: the head's selection rows (per query block, or per position of its group).  sink() takes the row
// constants, the selection and the row's Q and dO when do_rows asks for them.  Returns whether every dQ of the tile is finite.
// CAREFUL: tile by tile, with the elements that are not finite taken out.
template <typename T, int D, int BK, bool PERPOS, bool CAREFUL, typename TileRows, typename Sink>
__device__ __forceinline__ bool query_tile(const KParams &p, int I, int T0, int NT, int p0, int lane, const QueryHead &in,
                                           const TileRows &Kr, const TileRows &Vr, const int *sel_head, unsigned *my_lds,
                                           GateSums<D> &gate, const LaneMasks &lm, bool do_rows, bool do_dq, T *dQ_head, Sink &&sink)
{
  constexpr int CPL = Geo<D>::CPL, NMB = Geo<D>::NMB, NACC = Geo<D>::NACC;
  constexpr bool kDiag = kDiagonals<D, PERPOS>;
  const int q = lane & 15, g = lane >> 4;
  const float c2 = p.scale * kLog2eF, kc = Operands<T, D>::kBf ? c2 : 1.0f;  // (kc: what a product of rows is still to be multiplied by)
  const int iq = I * kTile + q;
  const bool active = iq < p.L && iq >= p0;
  using Ops = Operands<T, D>;
  typename Ops::Row qf, g_op;
  float gr[CPL], ol[CPL], os[CPL], wl[CPL], ws[CPL];
  gate.weights(g, wl, ws);
  const unsigned e_at = active ? (unsigned)(iq * D + CPL * g) : kNowhere / 4;  // rows that take no part read zeros
  load_op<T, D>(in.dO, e_at * (unsigned)sizeof(T), g_op);
  load_n<float>(in.o_lt, e_at * 4u, ol);
  load_n<float>(in.o_st, e_at * 4u, os);
  load_op<T, D>(in.Q, e_at * (unsigned)sizeof(T), qf);
  const unsigned l_at = active ? 4u * (unsigned)iq : kNowhere;
  float l2_lt = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(in.lse_lt.d, l_at, 0, 0)) * kLog2eF;
  float l2_st = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(in.lse_st.d, l_at, 0, 0)) * kLog2eF;
  if (!active) l2_lt = l2_st = kHugeF;
  LtSel<BK, PERPOS> ls;
  if constexpr (PERPOS) {
    int first[LtSel<BK, PERPOS>::kFirst];
    ls.request(p, sel_head, I, iq, lane, first);
    ls.build(p, my_lds, nullptr, sel_head + (size_t)min(iq, p.L - 1) * p.k, active, I, iq, p0, lane, first);
  } else {
    ls.build(p, my_lds, sel_head + (size_t)I * (kTile / BK) * p.k, I, p0, lane);
  }

  // ---- gate pass of the tile's rows ----
  Ops::floats(g_op, gr);
  const float a_ll = sum_g(dot_n(gr, ol, 0.0f)), a_ss = sum_g(dot_n(gr, os, 0.0f));
  const float w_l = sum_g(dot_n(wl, ol, 0.0f)), w_s = sum_g(dot_n(ws, os, 0.0f));
  float al = sigmoid(gate.bias + w_l + w_s);
  float dz = (a_ll - a_ss) * al * (1.0f - al);
  float D_lt = al * a_ll + dz * w_l, D_st = (1.0f - al) * a_ss + dz * w_s;
  if (!active) al = dz = D_lt = D_st = 0.0f;
  if (do_rows) {
    sink(I, al, dz, D_lt, D_st, l2_lt, l2_st, ls, qf, g_op);
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
      gate.gl[i] = fmaf(dz, ol[i], gate.gl[i]);
      gate.gs[i] = fmaf(dz, os[i], gate.gs[i]);
    }
    gate.gb += dz;
  }
  if (!do_dq) return true;

  Ops::scale(qf, c2);
#pragma unroll
  for (int i = 0; i < CPL; ++i) {
    ol[i] = fmaf(al, gr[i], dz * wl[i]);         // dO_lt of this lane's row
    os[i] = fmaf(1.0f - al, gr[i], dz * ws[i]);  // dO_st
  }
  const typename Ops::Split gl_op = Ops::split(ol), gs_op = Ops::split(os);
  f32x4 dq_part[NACC], dq[NMB];
  clear(dq_part);
  const int kid_q = mask_block(p, iq);
  const int J_hi = p.bidir ? NT - 1 : I;
  Walk wk;
  typename Ops::Row kf, vf;
  typename Ops::Col kt[NMB];
  auto products = [&](auto lt, auto st, f32x4 &s, f32x4 &g_lt, f32x4 &g_st) __attribute__((always_inline)) {
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    s = Ops::dot(kf, qf, zero);  // (times kc)
    if constexpr (decltype(lt)::value) g_lt = Ops::dot(vf, gl_op, zero);
    if constexpr (decltype(st)::value) g_st = Ops::dot(vf, gs_op, zero);
  };
  // did the lane's row select the tile, and is the key one that the causal and validity tests let through?
  auto selected = [&](int t) __attribute__((always_inline)) -> bool {
    bool x = wk.is_lt(t);
    if (PERPOS || BK < kTile) x &= ls.sees(q, t * kTile + 4 * g);
    return x;
  };
  const unsigned span = (unsigned)((p.bidir ? p.L - 1 : iq) - p0);
  auto seen = [&](int key) __attribute__((always_inline)) -> bool { return (unsigned)(key - p0) <= span; };
  auto add = [&](const float (&ds)[4]) __attribute__((always_inline)) { Ops::add(kt, ds, dq_part); };
  auto arg = [&](float s, float l) __attribute__((always_inline)) -> float { return Ops::kBf ? fmaf(kc, s, -l) : s - l; };
  auto body = [&](auto kind, auto unit, Word &mask) __attribute__((always_inline)) {
    constexpr int KIND = decltype(kind)::value;
    constexpr bool UNIT = decltype(unit)::value;
    const int t = wk.take(mask), t_next = wk.peek();
    f32x4 s, g_lt, g_st;
    products(std::bool_constant<KIND <= 1>{}, std::bool_constant<KIND != 1>{}, s, g_lt, g_st);
    Kr.op(t_next, kf);
    Vr.op(t_next, vf);
    const int key0 = t * kTile + 4 * g;
    float ds[4];
    if constexpr (KIND == 0) {
      const bool s_lt = selected(t);
      unsigned v_lt = 0u, v_st = 0u;
      if constexpr (UNIT) {
        const unsigned ok = LaneMasks::keys(p, key0, p0, iq);
        v_st = (lm.st<!kDiag>(p, I - t) | LaneMasks::from(p.last_lo - key0)) & ok;
        v_lt = s_lt ? ok : 0u;
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float e = __builtin_amdgcn_exp2f(arg(s[r], l2_lt)), f = __builtin_amdgcn_exp2f(arg(s[r], l2_st));
        if constexpr (UNIT) {
          e = keep(e, v_lt, r);
          f = keep(f, v_st, r);
        } else {
          const bool ok = seen(key0 + r);
          e = ok & s_lt ? e : 0.0f;
          f = ok & st_sees(p, iq, key0 + r, kid_q, mask_block(p, key0, r), key0 + r >= p.last_lo) ? f : 0.0f;
        }
        ds[r] = fmaf(f, g_st[r] - D_st, e * (g_lt[r] - D_lt));
      }
    } else if constexpr (KIND == 1) {
      const bool v = (PERPOS || BK < kTile) ? ls.sees(q, key0) : true;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float e = __builtin_amdgcn_exp2f(arg(s[r], l2_lt));
        ds[r] = ((PERPOS || BK < kTile) ? (v ? e : 0.0f) : e) * (g_lt[r] - D_lt);
      }
    } else {
      const unsigned v = UNIT ? lm.st<!kDiag>(p, I - t) : 0u;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float e = __builtin_amdgcn_exp2f(arg(s[r], l2_st));
        if constexpr (UNIT) e = keep(e, v, r);
        else e = st_sees(p, iq, key0 + r, kid_q, mask_block(p, key0, r), false) ? e : 0.0f;
        ds[r] = e * (g_st[r] - D_st);
      }
    }
    if constexpr (TileRows::kNear) Kr.col(t, kt);
    add(ds);
    if constexpr (!TileRows::kNear) Kr.col(t_next, kt);
  };
  auto word = [&](int w) __attribute__((always_inline)) {
    const int t = w * 64 + lane;
    const bool edge = (t == T0) | (t == I) | (t >= min(NT - 1, p.last_lo / kTile));
    wk.start<false>(p, I, w, T0, J_hi, lane, ls.has_tile(min(t, NT - 1)), edge, CAREFUL || !kDiag, true);
  };
  auto walk = [&](auto unit) __attribute__((always_inline)) {
    for (int w = T0 >> 6; w <= J_hi >> 6; ++w) {
      word(w);
      if (!wk.all()) continue;
      const int t = wk.peek();
      Kr.op(t, kf);
      Vr.op(t, vf);
      if constexpr (!TileRows::kNear) Kr.col(t, kt);
      while (wk.m0) body(std::integral_constant<int, 0>{}, unit, wk.m0);
      while (wk.m1) body(std::integral_constant<int, 1>{}, unit, wk.m1);
      while (wk.m2) body(std::integral_constant<int, 2>{}, unit, wk.m2);
    }
  };
  if constexpr (!CAREFUL) {
    auto far_keys = [&]() __attribute__((always_inline)) {
      float qd[CPL];
      Ops::floats(qf, qd);
      float qw[CPL * 4], ow[CPL * 4];
      if constexpr (D == 8) {
        whole_row(qd, qw);
        whole_row(os, ow);
      }
      diagonals(p, I, T0, J_hi, [&](int d) __attribute__((always_inline)) {
        if constexpr (D == 8) {
          const int t = min(max(I + d * (1 << g), T0), NT - 1), key = iq + kTile * d * (1 << g);
          float kr[D], vr[D];
          Kr.whole(t, kr);
          Vr.whole(t, vr);
          const float e = __builtin_amdgcn_exp2f(arg(dot_n(qw, kr, 0.0f), l2_st));
          const bool ok = (key >= p0) & (key < p.last_lo);
          add_row(dq_part, ok ? e * (dot_n(ow, vr, 0.0f) - D_st) : 0.0f, kr);
        } else {
        float s[4], x[4], ko[4][NMB][4];
#pragma unroll
        for (int n = 0; n < 4; ++n) {
          float kr[CPL], vr[CPL];
          const int t = min(max(I + d * (1 << n), T0), NT - 1);
          Kr.row(t, kr);
          Vr.row(t, vr);
          s[n] = dot_n(qd, kr, 0.0f);
          x[n] = dot_n(os, vr, 0.0f);
          if constexpr (D == 16) own_of_row(kr, ko[n]);
        }
        phase_end<D>();
        if constexpr (D != 16) {
#pragma unroll
          for (int n = 0; n < 4; ++n) Kr.own(min(max(I + d * (1 << n), T0), NT - 1), ko[n]);
        }
        const float e = __builtin_amdgcn_exp2f(arg(gather_g(s), l2_st)), gv = gather_g(x);
        const int key = iq + kTile * d * (1 << g);
        const bool ok = (key >= p0) & (key < p.last_lo);
        spread_g(ok ? e * (gv - D_st) : 0.0f, x);
        add_own(dq_part, x, ko);
        }
      });
    };
    if (kDiag && kFarFirst<D> && p.sblk == 1) far_keys();
    if (p.sblk <= 1) walk(std::true_type{});
    else walk(std::false_type{});
    if (kDiag && !kFarFirst<D> && p.sblk == 1) far_keys();
  } else {
    for (int w = T0 >> 6; w <= J_hi >> 6; ++w) {
      word(w);
      for (Word m = wk.all(); m;) {
        const int t = wk.take(m);
        Kr.op(t, kf);
        Vr.op(t, vf);
        Kr.col(t, kt);
        f32x4 s, g_lt, g_st;
        products(std::true_type{}, std::true_type{}, s, g_lt, g_st);
        float ds[4], lost[4];
        take_out<T, D>(kt, g, lost);
        const bool s_lt = selected(t);
        const int key0 = t * kTile + 4 * g;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const bool ok = seen(key0 + r);
          const bool v_st = ok & st_sees(p, iq, key0 + r, kid_q, mask_block(p, key0, r), key0 + r >= p.last_lo);
          const float e = __builtin_amdgcn_exp2f(arg(s[r], l2_lt)), f = __builtin_amdgcn_exp2f(arg(s[r], l2_st));
          ds[r] = ok & s_lt ? fmaf(e, g_lt[r] - D_lt, lost[r]) : 0.0f;
          ds[r] += v_st ? fmaf(f, g_st[r] - D_st, lost[r]) : 0.0f;
        }
        add(ds);
      }
    }
  }
  total<D>(dq_part, dq);
  const int el = fresh_lane(), ei = I * kTile + (el & 15);
  if (ei < p.L) store_grad_row<T, D>(dQ_head + (size_t)ei * D, dq, p.scale, ei >= p0, p, true, ei, el >> 4);
  return __all((ei < p0) | (ei >= p.L) | finite(abs_sum(dq)));
}

// Key tile J; kf, vf: this lane's channels of its key and value row (of the padding too, in the first tile with a valid
// row: a lane keeps to its own column, and those of the padding are stored as zeros).  The hpg query heads that read the
// rows add into the same gradients.  Returns whether all of them are finite; CAREFUL as above.  src gives their Q and dO rows, row constants, tile words and selection bits.
template <typename T, int D, int BK, bool PERPOS, bool CAREFUL, typename Src>
__device__ __forceinline__ bool key_tile(const KParams &p, int J, int T0, int NT, int p0, int lane, typename Operands<T, D>::Row &kf,
                                         const typename Operands<T, D>::Row &vf, int hpg, const Src &src, T *dK_head, T *dV_head)
{
  constexpr int CPL = Geo<D>::CPL, NMB = Geo<D>::NMB, NACC = Geo<D>::NACC;
  constexpr bool kDiag = kDiagonals<D, PERPOS>;
  const int q = lane & 15, g = lane >> 4;
  const int NWb = (p.NB + 31) / 32;
  using Ops = Operands<T, D>;
  const float c2 = p.scale * kLog2eF, kc = Ops::kBf ? c2 : 1.0f;  // (kc: what a product of rows is still to be multiplied by)
  const int j = J * kTile + q;
  f32x4 dk_part[NACC], dv_part[NACC];
  clear(dk_part);
  clear(dv_part);
  Ops::scale(kf, c2);
  const int kid_k = mask_block(p, j);
  const bool last_k = j >= p.last_lo;
  const int I_lo = p.bidir ? T0 : J;
  const int Jb = j / BK;  // this lane's key block
  const bool last_tile = J * kTile + kTile - 1 >= p.last_lo;  // holds last-block keys
  const LaneMasks lm = LaneMasks::make(p, q, g);

  for (int hl = 0; hl < hpg; ++hl) {
    const auto Qr = src.q_rows(hl);
    const auto Gr = src.g_rows(hl);
    constexpr bool near = decltype(src.q_rows(0))::kNear;
    const float *wrow = src.gate_row(hl);
    float t_lt = 0.0f, t_st = 0.0f;  // sum_i dz_i P_ij per branch
    float wv_lt, wv_st;              // Wg_x . v_j
    {
      float wl[CPL], ws[CPL], vd[CPL];
      Ops::floats(vf, vd);
      load_n<CPL>(wrow + CPL * g, wl);
      load_n<CPL>(wrow + D + CPL * g, ws);
      wv_lt = sum_g(dot_n(wl, vd, 0.0f));
      wv_st = sum_g(dot_n(ws, vd, 0.0f));
    }
    Walk wk;
    typename Ops::Row qa, ga;
    typename Ops::Col qc[NMB], gc[NMB];
    float al[4], dz[4], D_lt[4], D_st[4], l_lt[4], l_st[4];  // row constants of this lane's four query rows
    auto consts = [&](int I) __attribute__((always_inline)) {
      auto get = [&](int k, float (&x)[4]) { src.constant(hl, I, k, x); };
      get(0, al);
      get(1, dz);
      get(2, D_lt);
      get(3, D_st);
      get(4, l_lt);
      get(5, l_st);
    };
    auto products = [&](f32x4 &s, f32x4 &gv) __attribute__((always_inline)) {
      const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
      s = Ops::dot(qa, kf, zero);  // (times kc)
      gv = Ops::dot(ga, vf, zero);
    };
    auto arg = [&](float s, float l) __attribute__((always_inline)) -> float { return Ops::kBf ? fmaf(kc, s, -l) : s - l; };
    // bit 0 of w4[r]: row r of this lane's four of tile t selected this lane's key block
    auto selected = [&](int t, unsigned (&w4)[4]) __attribute__((always_inline)) {
      if constexpr (PERPOS) {
        const unsigned *sb = src.bits + (t * kTile + 4 * g) * 2 + (Jb >> 5);
#pragma unroll
        for (int r = 0; r < 4; ++r) w4[r] = sb[2 * r] >> (Jb & 31);
      } else if constexpr (BK < kTile) {
        const unsigned x = src.bits[(t * 2 + (g >> 1)) * NWb + min(Jb >> 5, NWb - 1)] >> (Jb & 31);
        w4[0] = w4[1] = w4[2] = w4[3] = x;
      }
    };
    // dV^T += dO^T (a P), dK^T += Q^T dS
    auto add = [&](const float (&pc)[4], const float (&ds)[4]) __attribute__((always_inline)) {
      Ops::add(gc, pc, dv_part);
      Ops::add(qc, ds, dk_part);
    };
    auto body = [&](auto kind, auto unit, Word &mask) __attribute__((always_inline)) {
      constexpr int KIND = decltype(kind)::value;
      constexpr bool LT = KIND <= 1, ST = KIND != 1, UNIT = decltype(unit)::value;
      const int t = wk.take(mask), t_next = wk.peek();
      if constexpr (near) consts(t);
      f32x4 s, gv;
      products(s, gv);
      Qr.op(t_next, qa);
      Gr.op(t_next, ga);
      const int i0 = t * kTile + 4 * g;  // this lane's rows i0 .. i0+3
      float pc[4], ds[4];
      unsigned w4[4] = {1u, 1u, 1u, 1u};
      if constexpr (LT) selected(t, w4);
      const bool in_lt = KIND != 0 || wk.is_lt(t);
      unsigned v_lt = 15u, v_st = 0u;  // UNIT: the masks as bits
      if constexpr (UNIT) {
        if constexpr (ST) v_st = lm.st<!kDiag>(p, J - t);
        if constexpr (KIND == 0) {
          const unsigned ok = LaneMasks::from(p.bidir ? 0 : j - i0);
          v_st = (last_k ? 15u : v_st) & ok;
          v_lt = in_lt ? ok : 0u;
        }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        bool ok = true;
        if constexpr (KIND == 0 && !UNIT) ok = (i0 + r >= j) | (p.bidir != 0);
        pc[r] = ds[r] = 0.0f;
        if constexpr (LT) {
          const float e = __builtin_amdgcn_exp2f(arg(s[r], l_lt[r]));
          float pr = e;
          if constexpr (KIND == 0 && UNIT) pr = keep(pr, v_lt, r);
          if constexpr (KIND == 0 && !UNIT) pr = ok & in_lt ? pr : 0.0f;
          if constexpr (PERPOS || BK < kTile) pr = keep(pr, w4[r], 0);
          pc[r] = al[r] * pr;
          ds[r] = pr * fmaf(al[r], gv[r], fmaf(dz[r], wv_lt, -D_lt[r]));
          t_lt = fmaf(dz[r], pr, t_lt);
        }
        if constexpr (ST) {
          const float e = __builtin_amdgcn_exp2f(arg(s[r], l_st[r]));
          float pr = e;
          if constexpr (UNIT) pr = keep(pr, v_st, r);
          else pr = ok & st_sees(p, i0 + r, j, mask_block(p, i0, r), kid_k, KIND == 0 ? last_k : false) ? pr : 0.0f;
          const float as = 1.0f - al[r];
          pc[r] = fmaf(as, pr, pc[r]);
          ds[r] = fmaf(pr, fmaf(as, gv[r], fmaf(dz[r], wv_st, -D_st[r])), ds[r]);
          t_st = fmaf(dz[r], pr, t_st);
        }
      }
      if constexpr (!near) {
        consts(t_next);
      } else {
        Qr.col(t, qc);
        Gr.col(t, gc);
      }
      add(pc, ds);
      if constexpr (!near) {
        Qr.col(t_next, qc);
        Gr.col(t_next, gc);
      }
    };
    auto word = [&](int w) __attribute__((always_inline)) {
      const int t = w * 64 + lane;
      const unsigned tw = src.tile_word(min(max(t, T0), NT - 1), J >> 5);
      wk.start<true>(p, J, w, I_lo, NT - 1, lane, (tw >> (J & 31)) & 1u, last_tile | (t == J), CAREFUL || !kDiag, true);
    };
    auto walk = [&](auto unit) __attribute__((always_inline)) {
      for (int w = I_lo >> 6; w <= (NT - 1) >> 6; ++w) {
        word(w);
        if (!wk.all()) continue;
        const int t = wk.peek();
        Qr.op(t, qa);
        Gr.op(t, ga);
        if constexpr (!near) {
          consts(t);
          Qr.col(t, qc);
          Gr.col(t, gc);
        }
        while (wk.m0) body(std::integral_constant<int, 0>{}, unit, wk.m0);
        while (wk.m1) body(std::integral_constant<int, 1>{}, unit, wk.m1);
        while (wk.m2) body(std::integral_constant<int, 2>{}, unit, wk.m2);
      }
    };
    auto walk_carefully = [&]() __attribute__((always_inline)) {
      for (int w = I_lo >> 6; w <= (NT - 1) >> 6; ++w) {
        word(w);
        for (Word m = wk.all(); m;) {
          const int t = wk.take(m);
          consts(t);
          Qr.op(t, qa);
          Gr.op(t, ga);
          Qr.col(t, qc);
          Gr.col(t, gc);
          f32x4 s, gv;
          products(s, gv);
          unsigned w4[4] = {1u, 1u, 1u, 1u};
          selected(t, w4);
          float lost_q[4], lost_g[4];
          take_out<T, D>(qc, g, lost_q);
          take_out<T, D>(gc, g, lost_g);
          const bool in_lt = wk.is_lt(t);
          float pc[4], ds[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int i = t * kTile + 4 * g + r;
            const bool ok = (i >= p0) & (i < p.L) & ((i >= j) | (p.bidir != 0));
            const bool v_lt = ok & in_lt & ((w4[r] & 1u) != 0u);
            const bool v_st = ok & st_sees(p, i, j, mask_block(p, i), kid_k, last_k);
            const float e = __builtin_amdgcn_exp2f(arg(s[r], l_lt[r])), f = __builtin_amdgcn_exp2f(arg(s[r], l_st[r]));
            const float as = 1.0f - al[r];
            pc[r] = v_lt ? fmaf(al[r], e, lost_g[r]) : 0.0f;
            pc[r] += v_st ? fmaf(as, f, lost_g[r]) : 0.0f;
            ds[r] = v_lt ? fmaf(e, fmaf(al[r], gv[r], fmaf(dz[r], wv_lt, -D_lt[r])), lost_q[r]) : 0.0f;
            ds[r] += v_st ? fmaf(f, fmaf(as, gv[r], fmaf(dz[r], wv_st, -D_st[r])), lost_q[r]) : 0.0f;
            t_lt += v_lt ? dz[r] * e : 0.0f;
            t_st += v_st ? dz[r] * f : 0.0f;
          }
          add(pc, ds);
        }
      }
    };
    auto far_queries = [&]() __attribute__((always_inline)) {
      float kd[CPL], vd[CPL];
      Ops::floats(kf, kd);
      Ops::floats(vf, vd);
      float kw[CPL * 4], vw[CPL * 4];
      if constexpr (D == 8) {
        whole_row(kd, kw);
        whole_row(vd, vw);
      }
      diagonals(p, J, I_lo, NT - 1, [&](int d) __attribute__((always_inline)) {
        // this lane group's distance
        const int i = j + kTile * d * (1 << g), tg = min(max(J + d * (1 << g), I_lo), NT - 1);
        auto constant = [&](int k) { return src.row_constant(hl, tg, k); };
        const bool ok = (i >= p0) & (i < p.L) & !last_k;
        if constexpr (D == 8) {
          float qr[D], gr[D];
          Qr.whole(tg, qr);
          Gr.whole(tg, gr);
          const float e = __builtin_amdgcn_exp2f(arg(dot_n(kw, qr, 0.0f), constant(5)));
          const float pr = ok ? e : 0.0f, zd = constant(1), as = 1.0f - constant(0);
          t_st = fmaf(zd, pr, t_st);
          add_row(dv_part, as * pr, gr);
          add_row(dk_part, pr * fmaf(as, dot_n(vw, gr, 0.0f), fmaf(zd, wv_st, -constant(3))), qr);
        } else {
        float s[4], x[4], qo[4][NMB][4], go[4][NMB][4];
#pragma unroll
        for (int n = 0; n < 4; ++n) {
          float qr[CPL], gr[CPL];
          const int t = min(max(J + d * (1 << n), I_lo), NT - 1);
          Qr.row(t, qr);
          Gr.row(t, gr);
          s[n] = dot_n(kd, qr, 0.0f);
          x[n] = dot_n(vd, gr, 0.0f);
          if constexpr (D == 16) {
            own_of_row(qr, qo[n]);
            own_of_row(gr, go[n]);
          }
        }
        phase_end<D>();
        if constexpr (D != 16) {
#pragma unroll
          for (int n = 0; n < 4; ++n) {
            const int t = min(max(J + d * (1 << n), I_lo), NT - 1);
            Qr.own(t, qo[n]);
            Gr.own(t, go[n]);
          }
        }
        const float e = __builtin_amdgcn_exp2f(arg(gather_g(s), constant(5))), gd = gather_g(x);
        const float pr = ok ? e : 0.0f;
        const float zd = constant(1), as = 1.0f - constant(0);
        t_st = fmaf(zd, pr, t_st);
        spread_g(as * pr, s);
        spread_g(pr * fmaf(as, gd, fmaf(zd, wv_st, -constant(3))), x);
        add_own(dv_part, s, go);
        add_own(dk_part, x, qo);
        }
      });
    };
    if constexpr (CAREFUL) {
      walk_carefully();
    } else {
      if (kDiag && kFarFirst<D> && p.sblk == 1) far_queries();
      if (p.sblk <= 1) walk(std::true_type{});
      else walk(std::false_type{});
      if (kDiag && !kFarFirst<D> && p.sblk == 1) far_queries();
    }
    // the gate part of dV: sum_i dz_i P_ij times the gate row of the branch
    if constexpr (Geo<D>::kQuads) {  // (a lane's part of the sums, like the accumulators)
#pragma unroll
      for (int h = 0; h < NACC; ++h) {
        float x[4], y[4];
        load_n<4>(wrow + 4 * h, x);
        load_n<4>(wrow + D + 4 * h, y);
#pragma unroll
        for (int r = 0; r < 4; ++r) dv_part[h][r] += fmaf(t_lt, x[r], t_st * y[r]);
      }
    } else {
      t_lt = sum_g(t_lt);
      t_st = sum_g(t_st);
#pragma unroll
      for (int mb = 0; mb < NMB; ++mb) {
        float x[4], y[4];
        load_n<4>(wrow + 16 * mb + 4 * g, x);
        load_n<4>(wrow + D + 16 * mb + 4 * g, y);
#pragma unroll
        for (int r = 0; r < 4; ++r) dv_part[mb][r] += fmaf(t_lt, x[r], t_st * y[r]);
      }
    }
  }
  f32x4 dk[NMB], dv[NMB];
  total<D>(dk_part, dk);
  total<D>(dv_part, dv);
  const int el = fresh_lane(), ej = J * kTile + (el & 15);
  if (ej < p.L) {
    store_grad_row<T, D>(dK_head + (size_t)ej * D, dk, p.scale, ej >= p0, p, true, ej, el >> 4);
    store_grad_row<T, D>(dV_head + (size_t)ej * D, dv, 1.0f, ej >= p0, p, false, ej, el >> 4);
  }
  return __all((ej < p0) | (ej >= p.L) | finite(abs_sum(dk) + abs_sum(dv)));
}

// A wavefront's query tiles again, for one of which dQ was not finite.  Out of the loop over the tiles and with everything read
// anew: beside the walk this code took registers from it (a training step at B=32 H=8 L=2000 d=8 375 us, 358 like this).
template <typename T, int D, int BK, bool PERPOS>
__device__ __forceinline__ void query_tiles_carefully(const KParams &p, int first, int step, int T0, int NT, int p0, int lane,
                                                      const QueryHead &in, const Rows<T, D> &Kr, const Rows<T, D> &Vr, const int *sel_head,
                                                      unsigned *my_lds, const float *gate_w, const float *gate_b, int h, T *dQ_head)
{
  GateSums<D> gate(gate_w, gate_b, h);
  const LaneMasks lm{};
  for (int u = first; u < NT - T0; u += step)
    query_tile<T, D, BK, PERPOS, true>(p, NT - 1 - u, T0, NT, p0, lane, in, Kr, Vr, sel_head, my_lds, gate, lm, false, true, dQ_head,
                                       [](auto &&...) {});
}

// The gate gradient sums of a head's rows that a wavefront takes, in registers until leave().  d = 32: the walk needs the seventeen
// registers, so every tile's sums over its rows go to LDS at once (mine[2D + 1], cleared by the caller): spilled registers in bf16 18 -> 1,
// with two blocks to a tile in fp32 53 -> 20, a whole training step at B=180 H=4 L=150 d=32 b=8 fp32 98.5 us with them in registers, 89.2 so.
template <int D>
struct NearGateSums {
  static constexpr int CPL = Geo<D>::CPL;
  static constexpr bool kInLds = D == 32;
  float bias, *mine, gl[kInLds ? 1 : CPL], gs[kInLds ? 1 : CPL], gb;
  __device__ __forceinline__ NearGateSums(const float *gate_b, int h, float *mine_) : bias(gate_b ? gate_b[h] : 0.0f), mine(mine_)
  {
    zero_n(gl);
    zero_n(gs);
    gb = 0.0f;
  }
  __device__ __forceinline__ void add(float dz, const float (&ol)[CPL], const float (&os)[CPL], int lane)
  {
    if constexpr (kInLds) {
      const int q = lane & 15, g = lane >> 4;
      float x[CPL], y[CPL];
#pragma unroll
      for (int i = 0; i < CPL; ++i) {
        x[i] = sum_row(dz * ol[i]);
        y[i] = sum_row(dz * os[i]);
      }
      const float z = sum_row(dz);
      if (q == 0) {
#pragma unroll
        for (int i = 0; i < CPL; ++i) {
          mine[CPL * g + i] += x[i];
          mine[D + CPL * g + i] += y[i];
        }
        if (g == 0) mine[2 * D] += z;
      }
    } else {
#pragma unroll
      for (int i = 0; i < CPL; ++i) {
        gl[i] = fmaf(dz, ol[i], gl[i]);
        gs[i] = fmaf(dz, os[i], gs[i]);
      }
      gb += dz;
    }
  }
  __device__ __forceinline__ void leave(int lane)
  {
    if constexpr (!kInLds) {
      const int q = lane & 15, g = lane >> 4;
#pragma unroll
      for (int i = 0; i < CPL; ++i) {
        gl[i] = sum_row(gl[i]);
        gs[i] = sum_row(gs[i]);
      }
      gb = sum_row(gb);
      if (q == 0) {
#pragma unroll
        for (int i = 0; i < CPL; ++i) {
          mine[CPL * g + i] = gl[i];
          mine[D + CPL * g + i] = gs[i];
        }
        if (g == 0) mine[2 * D] = gb;
      }
    }
  }
};

// THE NEAR FORM of the two (see there).  What a query tile needs from memory, requested a tile ahead.
template <typename T, int D, int BK, bool PERPOS>
struct QueryIn {
  using Ops = Operands<T, D>;
  typename Ops::Row q, g;
  float ol[Geo<D>::CPL], os[Geo<D>::CPL], lse[2];
  int sel[LtSel<BK, PERPOS>::kFirst];
  // (d = 32: 27 or 35 registers, which the walk needs; the request goes out between the walk and the stores)
  static constexpr bool kEarly = D < 32;
  // any: is there such a tile?  (Nothing is read when there is none, but the registers are written: a request under a branch would
  // keep what they held alive through the walk before it.)
  __device__ __forceinline__ void request(const KParams &p, int I, int p0, int lane, const QueryHead &in, const int *sel_head, bool any)
  {
    I = any ? I : 0;
    const int iq = I * kTile + (lane & 15);
    const bool active = any & (iq < p.L) & (iq >= p0);
    const unsigned at = active ? (unsigned)(iq * D + Geo<D>::CPL * (lane >> 4)) : kNowhere / 4;  // rows that take no part read zeros
    load_op<T, D>(in.dO, at * (unsigned)sizeof(T), g);
    load_n<float>(in.o_lt, at * 4u, ol);
    load_n<float>(in.o_st, at * 4u, os);
    load_op<T, D>(in.Q, at * (unsigned)sizeof(T), q);
    const unsigned l_at = active ? 4u * (unsigned)iq : kNowhere;
    lse[0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(in.lse_lt.d, l_at, 0, 0));
    lse[1] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(in.lse_st.d, l_at, 0, 0));
    LtSel<BK, PERPOS>::request(p, sel_head, I, iq, lane, sel);
    asm volatile("" ::: "memory");
  }
  // Waits for them: before a tile's stores go out, for behind those a wait for them would be one for the stores.
  __device__ __forceinline__ void arrived()
  {
    Ops::arrived(q);
    Ops::arrived(g);
    arrive(ol);
    arrive(os);
    arrive(lse);
    arrive(sel);
  }
};

// Query tile I, whose rows are in `x`; more(x) requests the next one's there.  w_gate: the head's gate row in LDS.  sink: as in
// query_tile, with the long-term tiles (tiles_of(word)) beside the selection.
template <typename T, int D, int BK, bool PERPOS, bool ONE_WORD, typename TileRows, typename More, typename Sink>
__device__ __forceinline__ bool near_query_tile(const KParams &p, int I, int T0, int NT, int p0, int lane, QueryIn<T, D, BK, PERPOS> &x,
                                                const TileRows &Kr, const TileRows &Vr, const int *sel_head, unsigned *my_lds,
                                                const float *w_gate, NearGateSums<D> &gate, const NearMasks &nm, const Word (&valid_keys)[4],
                                                bool do_rows, bool do_dq, T *dQ_head, More &&more, Sink &&sink, float *turn = nullptr)
{
  constexpr int CPL = Geo<D>::CPL, NMB = Geo<D>::NMB, NACC = Geo<D>::NACC;
  constexpr bool kDiag = kDiagonals<D, PERPOS>, kPicked = !PERPOS && BK == kTile;
  using Ops = Operands<T, D>;
  using Sel = LtSel<BK, PERPOS>;
  const int q = lane & 15, g = lane >> 4;
  const float c2 = p.scale * kLog2eF, kc = Ops::kBf ? c2 : 1.0f;  // (kc: what a product of rows is still to be multiplied by)
  const int iq = I * kTile + q;
  const bool active = iq < p.L && iq >= p0;
  typename Ops::Row qf = x.q, g_op = x.g;
  float ol[CPL], os[CPL], gr[CPL], wl[CPL], ws[CPL];
  int first[Sel::kFirst];
#pragma unroll
  for (int i = 0; i < CPL; ++i) {
    ol[i] = x.ol[i];
    os[i] = x.os[i];
  }
#pragma unroll
  for (int i = 0; i < Sel::kFirst; ++i) first[i] = x.sel[i];
  const float l2_lt = active ? x.lse[0] * kLog2eF : kHugeF, l2_st = active ? x.lse[1] * kLog2eF : kHugeF;
  if constexpr (QueryIn<T, D, BK, PERPOS>::kEarly) more(x);
  load_n<CPL>(w_gate + CPL * g, wl);
  load_n<CPL>(w_gate + D + CPL * g, ws);
  Sel ls;
  if constexpr (!kPicked)
    ls.build(p, my_lds, PERPOS ? nullptr : sel_head + (size_t)I * (kTile / BK) * p.k, sel_head + (size_t)min(iq, p.L - 1) * p.k, active, I, iq,
             p0, lane, first);
  auto tiles_of = [&](int w) __attribute__((always_inline)) -> Word {
    if constexpr (kPicked) return PickedTiles{sel_head + (size_t)I * p.k, p.k, first[0]}.word(w, lane);
    else if constexpr (PERPOS) return ls.all;
    else return __ballot(ls.has_tile(min(w * 64 + lane, NT - 1)));
  };

  // ---- gate pass of the tile's rows ----
  Ops::floats(g_op, gr);
  float al, dz, D_lt, D_st;
  {
    const float part[4] = {dot_n(gr, ol, 0.0f), dot_n(gr, os, 0.0f), dot_n(wl, ol, 0.0f), dot_n(ws, os, 0.0f)};
    float sum[4];  // dO.o_lt, dO.o_st, Wg_lt.o_lt, Wg_st.o_st
    spread_g(gather_g(part), sum);
    al = sigmoid(gate.bias + sum[2] + sum[3]);
    dz = (sum[0] - sum[1]) * al * (1.0f - al);
    D_lt = al * sum[0] + dz * sum[2];
    D_st = (1.0f - al) * sum[1] + dz * sum[3];
  }
  if (!active) al = dz = D_lt = D_st = 0.0f;
  const int w0 = ONE_WORD ? 0 : T0 >> 6, wI = ONE_WORD ? 0 : I >> 6;
  const Word at_I = tiles_of(wI);
  if (do_rows) {
    sink(I, al, dz, D_lt, D_st, l2_lt, l2_st, ls, qf, g_op, [&](int w) __attribute__((always_inline)) { return w == wI ? at_I : tiles_of(w); });
    gate.add(dz, ol, os, lane);
  }
  if (!do_dq) return true;

  Ops::scale(qf, c2);
#pragma unroll
  for (int i = 0; i < CPL; ++i) {
    ol[i] = fmaf(al, gr[i], dz * wl[i]);         // dO_lt of this lane's row
    os[i] = fmaf(1.0f - al, gr[i], dz * ws[i]);  // dO_st
  }
  const typename Ops::Split gl_op = Ops::split(ol), gs_op = Ops::split(os);
  f32x4 dq_part[NACC], dq[NMB];
  clear(dq_part);
  typename Ops::Row kf, vf;
  typename Ops::Col kt[NMB];
  auto arg = [&](float s, float l) __attribute__((always_inline)) -> float { return Ops::kBf ? fmaf(kc, s, -l) : s - l; };
  auto tile = [&](auto lt, auto st, auto masked, int t, int t_next, const Word (&m_lt)[4], const Word (&m_st)[4])
                  __attribute__((always_inline)) {
    constexpr bool LT = decltype(lt)::value, ST = decltype(st)::value, MASKED = decltype(masked)::value;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    if constexpr (!TileRows::kNear) LdsRows<T, D>::put(turn, q, g, kf);
    const f32x4 s = Ops::dot(kf, qf, zero);  // (times kc)
    f32x4 g_lt, g_st;
    if constexpr (LT) g_lt = Ops::dot(vf, gl_op, zero);
    if constexpr (ST) g_st = Ops::dot(vf, gs_op, zero);
    Kr.op(t_next, kf);
    Vr.op(t_next, vf);
    bool mine = true;
    if constexpr (LT && (PERPOS || BK < kTile)) mine = ls.sees(q, t * kTile + 4 * g);
    float ds[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      ds[r] = 0.0f;
      if constexpr (LT) {
        const float e = __builtin_amdgcn_exp2f(arg(s[r], l2_lt));
        ds[r] = (mine && (!MASKED || in_lanes(m_lt[r])) ? e : 0.0f) * (g_lt[r] - D_lt);
      }
      if constexpr (ST) {
        const float f = __builtin_amdgcn_exp2f(arg(s[r], l2_st)), fm = in_lanes(m_st[r]) ? f : 0.0f;
        ds[r] = LT ? fmaf(fm, g_st[r] - D_st, ds[r]) : fm * (g_st[r] - D_st);
      }
    }
    if constexpr (TileRows::kNear) Kr.col(t, kt);
    else LdsRows<T, D>(turn, q, g).col(0, kt);
    Ops::add(kt, ds, dq_part);
  };
  auto walk = [&]() __attribute__((always_inline)) {
    constexpr auto yes = std::true_type{};
    constexpr auto no = std::false_type{};
    auto request = [&](int t) __attribute__((always_inline)) {
      Kr.op(t, kf);
      Vr.op(t, vf);
    };
    const bool own = (at_I >> (I & 63)) & 1ull;
    const bool before = (wI != w0 && (I & 63) == 0 ? tiles_of(wI - 1) : at_I) >> ((I - 1) & 63) & 1ull;
    // of word w, the tiles from the first valid one to the last but one before I
    auto rest_of = [&](int w) __attribute__((always_inline)) -> Word {
      Word m = w == wI ? at_I : tiles_of(w);
      if (w == w0) m &= ~0ull << (T0 & 63);
      if (w == (I - 1) >> 6) m &= (1ull << ((I - 1) & 63)) - 1ull;
      return w > (I - 1) >> 6 ? 0ull : m;
    };
    Word rest = I > T0 ? rest_of(w0) : 0ull;
    auto next_of = [&](int w, Word m) __attribute__((always_inline)) -> int { return m ? 64 * w + __builtin_ctzll(m) : max(I - 1, T0); };
    // The long-term tiles, the tile before, the own one: small terms first.  The other way round dQ errs more against 64 bits than in
    // query_tile, 1.03 times as much in the mean at d = 16 and 32 and up to 1.07; so 0.95 and 0.96, 0.98 at d = 8.
    Word m_lt[4], m_st[4];
    if (kDiag || p.sblk != 1 || I - 2 < T0) request(next_of(w0, rest));
    if constexpr (!kDiag) {  // (per position: a single word)
      if (p.sblk == 1)
        for (int d = 2; I - d >= T0; d *= 2) {
          const int t = I - d;
          const bool here = (rest >> (t & 63)) & 1ull;
          rest &= ~(1ull << (t & 63));
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            m_lt[r] = t == T0 ? valid_keys[r] : ~0ull;
            m_st[r] = triangle(r, false) & triangle(r, true) & m_lt[r];
          }
          if (TileRows::kNear || d == 2) request(t);
          const int t_next = I - 2 * d >= T0 ? I - 2 * d : next_of(w0, rest);
          if (here) tile(yes, yes, yes, t, t_next, m_lt, m_st);
          else tile(no, yes, yes, t, t_next, m_lt, m_st);
        }
    }
    for (int w = w0;;) {
      if (w == w0 && (rest >> (T0 & 63)) & 1ull) {
        rest &= rest - 1;
        tile(yes, no, yes, T0, next_of(w, rest), valid_keys, valid_keys);
      }
      while (rest) {
        const int t = 64 * w + __builtin_ctzll(rest);
        rest &= rest - 1;
        tile(yes, no, no, t, next_of(w, rest), m_lt, m_st);
      }
      if (ONE_WORD || ++w > wI) break;
      rest = rest_of(w);
      request(next_of(w, rest));
    }
    if (I > T0) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        m_lt[r] = I - 1 == T0 ? valid_keys[r] : ~0ull;
        m_st[r] = nm.next[r] & m_lt[r];
      }
      if (before) tile(yes, yes, yes, I - 1, I, m_lt, m_st);
      else tile(no, yes, yes, I - 1, I, m_lt, m_st);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const Word ok = I == T0 ? valid_keys[r] : ~0ull;
      m_lt[r] = own ? triangle(r, false) & ok : 0ull;
      m_st[r] = nm.own[r] & ok;
    }
    tile(yes, yes, yes, I, I, m_lt, m_st);
  };
  auto far_keys = [&]() __attribute__((always_inline)) {
    float qd[CPL];
    Ops::floats(qf, qd);
    float qw[CPL * 4], ow[CPL * 4];
    if constexpr (D == 8) {
      whole_row(qd, qw);
      whole_row(os, ow);
    }
    diagonals(p, I, T0, I, [&](int d) __attribute__((always_inline)) {
      const bool ok = iq + kTile * d * (1 << g) >= p0;
      if constexpr (D == 8) {
        const int t = max(I + d * (1 << g), T0);
        float kr[D], vr[D];
        Kr.whole(t, kr);
        Vr.whole(t, vr);
        const float e = __builtin_amdgcn_exp2f(arg(dot_n(qw, kr, 0.0f), l2_st));
        add_row(dq_part, ok ? e * (dot_n(ow, vr, 0.0f) - D_st) : 0.0f, kr);
      } else {
        float s[4], y[4], ko[4][NMB][4];
#pragma unroll
        for (int n = 0; n < 4; ++n) {
          float kr[CPL], vr[CPL];
          const int t = max(I + d * (1 << n), T0);
          Kr.row(t, kr);
          Vr.row(t, vr);
          s[n] = dot_n(qd, kr, 0.0f);
          y[n] = dot_n(os, vr, 0.0f);
          if constexpr (D == 16) own_of_row(kr, ko[n]);
        }
        phase_end<D>();
        if constexpr (D != 16) {
#pragma unroll
          for (int n = 0; n < 4; ++n) Kr.own(max(I + d * (1 << n), T0), ko[n]);
        }
        const float e = __builtin_amdgcn_exp2f(arg(gather_g(s), l2_st)), gv = gather_g(y);
        spread_g(ok ? e * (gv - D_st) : 0.0f, y);
        add_own(dq_part, y, ko);
      }
    });
  };
  if (kDiag && kFarFirst<D> && p.sblk == 1) far_keys();
  walk();
  if (kDiag && !kFarFirst<D> && p.sblk == 1) far_keys();
  total<D>(dq_part, dq);
  if constexpr (QueryIn<T, D, BK, PERPOS>::kEarly) x.arrived();
  else more(x);
  const int el = fresh_lane(), ei = I * kTile + (el & 15);
  if (ei < p.L) store_grad_row<T, D>(dQ_head + (unsigned)ei * D, dq, p.scale, ei >= p0, p, true, ei, el >> 4);
  return __ballot(!((ei < p0) | (ei >= p.L) | finite(abs_sum(dq)))) == 0ull;
}

// Key tile J; its rows in kf, vf as in key_tile.  more() requests the next tile's rows, arrived() waits for them before the stores.
template <typename T, int D, int BK, bool PERPOS, bool ONE_WORD, typename Src, typename More, typename Arrived>
__device__ __forceinline__ bool near_key_tile(const KParams &p, int J, int T0, int NT, int p0, int lane, typename Operands<T, D>::Row kf,
                                              const typename Operands<T, D>::Row vf, int hpg, const Src &src, const NearMasks &nm, T *dK_head,
                                              T *dV_head, More &&more, Arrived &&arrived, float *turn = nullptr)
{
  constexpr int CPL = Geo<D>::CPL, NMB = Geo<D>::NMB, NACC = Geo<D>::NACC;
  constexpr bool kDiag = kDiagonals<D, PERPOS>;
  using Ops = Operands<T, D>;
  const int q = lane & 15, g = lane >> 4;
  const int NWb = (p.NB + 31) / 32;
  const float c2 = p.scale * kLog2eF, kc = Ops::kBf ? c2 : 1.0f;  // (kc: what a product of rows is still to be multiplied by)
  const int j = J * kTile + q;
  f32x4 dk_part[NACC], dv_part[NACC];
  clear(dk_part);
  clear(dv_part);
  Ops::scale(kf, c2);
  const int Jb = j / BK;  // this lane's key block
  // the query tiles of word w, from J on, that selected the tile
  const int wJ = ONE_WORD ? 0 : J >> 6, wE = ONE_WORD ? 0 : (NT - 1) >> 6;
  auto tiles_of = [&](int w) __attribute__((always_inline)) -> Word {
    const int t = w * 64 + lane;
    const unsigned tw = src.tile_word(min(max(t, T0), NT - 1), J >> 5);
    return __ballot((t >= J) & (t < NT) & ((tw >> (J & 31)) & 1u));
  };
  const Word at_J = tiles_of(wJ);
  constexpr bool kEarly = D < 32;
  if constexpr (kEarly) more();

  for (int hl = 0; hl < hpg; ++hl) {
    const auto Qr = src.q_rows(hl);
    const auto Gr = src.g_rows(hl);
    constexpr bool near = decltype(src.q_rows(0))::kNear;
    const float *wrow = src.gate_row(hl);
    float t_lt = 0.0f, t_st = 0.0f;  // sum_i dz_i P_ij per branch
    float wv_lt, wv_st;              // Wg_x . v_j
    {
      float wl[CPL], ws[CPL], vd[CPL];
      Ops::floats(vf, vd);
      load_n<CPL>(wrow + CPL * g, wl);
      load_n<CPL>(wrow + D + CPL * g, ws);
      wv_lt = sum_g(dot_n(wl, vd, 0.0f));
      wv_st = sum_g(dot_n(ws, vd, 0.0f));
    }
    typename Ops::Row qa, ga;
    typename Ops::Col qc[NMB], gc[NMB];
    float al[4], dz[4], D_lt[4], D_st[4], l_lt[4], l_st[4];  // row constants of this lane's four query rows
    // streamed: the tiles' rows go through this wavefront's part of LDS (see turn_floats), the constants 16 bytes a lane
    constexpr int kTurn = kTile * kLdsRow<T, D>;
    float raw[4] = {0.f, 0.f, 0.f, 0.f};
    auto consts = [&](int I) __attribute__((always_inline)) {
      auto get = [&](int k, float (&x)[4]) {
        if constexpr (near) src.constant(hl, I, k, x);
        else load_n<4>(turn + 2 * kTurn + 16 * k + 4 * g, x);
      };
      get(0, al);
      get(1, dz);
      get(2, D_lt);
      get(3, D_st);
      get(4, l_lt);
      get(5, l_st);
    };
    auto arg = [&](float s, float l) __attribute__((always_inline)) -> float { return Ops::kBf ? fmaf(kc, s, -l) : s - l; };
    auto tile = [&](auto lt, auto st, auto masked, int t, int t_next, const Word (&m_lt)[4], const Word (&m_st)[4])
                    __attribute__((always_inline)) {
      constexpr bool LT = decltype(lt)::value, ST = decltype(st)::value, MASKED = decltype(masked)::value;
      if constexpr (!near) {
        LdsRows<T, D>::put(turn, q, g, qa);
        LdsRows<T, D>::put(turn + kTurn, q, g, ga);
        if (lane < 24) store_lds(turn + 2 * kTurn + 4 * lane, raw);
      }
      consts(t);
      const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
      const f32x4 s = Ops::dot(qa, kf, zero), gv = Ops::dot(ga, vf, zero);  // (s: times kc)
      Qr.op(t_next, qa);
      Gr.op(t_next, ga);
      if constexpr (!near) src.constants(hl, t_next, lane, raw);
      unsigned w4[4] = {1u, 1u, 1u, 1u};  // bit 0: the row selected this lane's key block
      if constexpr (LT && PERPOS) {
        const unsigned *sb = src.bits + (t * kTile + 4 * g) * 2 + (Jb >> 5);
#pragma unroll
        for (int r = 0; r < 4; ++r) w4[r] = sb[2 * r] >> (Jb & 31);
      } else if constexpr (LT && BK < kTile) {
        const unsigned x = src.bits[(t * 2 + (g >> 1)) * NWb + min(Jb >> 5, NWb - 1)] >> (Jb & 31);
        w4[0] = w4[1] = w4[2] = w4[3] = x;
      }
      float pc[4], ds[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        pc[r] = ds[r] = 0.0f;
        if constexpr (LT) {
          float pr = __builtin_amdgcn_exp2f(arg(s[r], l_lt[r]));
          if constexpr (MASKED) pr = in_lanes(m_lt[r]) ? pr : 0.0f;
          if constexpr (PERPOS || BK < kTile) pr = keep(pr, w4[r], 0);
          pc[r] = al[r] * pr;
          ds[r] = pr * fmaf(al[r], gv[r], fmaf(dz[r], wv_lt, -D_lt[r]));
          t_lt = fmaf(dz[r], pr, t_lt);
        }
        if constexpr (ST) {
          const float e = __builtin_amdgcn_exp2f(arg(s[r], l_st[r])), pr = in_lanes(m_st[r]) ? e : 0.0f;
          const float as = 1.0f - al[r], x = fmaf(as, gv[r], fmaf(dz[r], wv_st, -D_st[r]));
          pc[r] = LT ? fmaf(as, pr, pc[r]) : as * pr;
          ds[r] = LT ? fmaf(pr, x, ds[r]) : pr * x;
          t_st = fmaf(dz[r], pr, t_st);
        }
      }
      if constexpr (near) {
        Qr.col(t, qc);
        Gr.col(t, gc);
      } else {
        LdsRows<T, D>(turn, q, g).col(0, qc);
        LdsRows<T, D>(turn + kTurn, q, g).col(0, gc);
      }
      Ops::add(gc, pc, dv_part);  // dV^T += dO^T (a P), dK^T += Q^T dS
      Ops::add(qc, ds, dk_part);
    };
    auto request = [&](int t) __attribute__((always_inline)) {
      Qr.op(t, qa);
      Gr.op(t, ga);
      if constexpr (!near) src.constants(hl, t, lane, raw);
    };
    auto walk = [&]() __attribute__((always_inline)) {
      constexpr auto yes = std::true_type{};
      constexpr auto no = std::false_type{};
      request(J);
      const bool own = (at_J >> (J & 63)) & 1ull;
      const bool after = (wE != wJ && ((J + 1) & 63) == 0 ? tiles_of(wJ + 1) : at_J) >> ((J + 1) & 63) & 1ull;
      // of word w, the tiles from the second after J on
      auto rest_of = [&](int w) __attribute__((always_inline)) -> Word {
        Word m = w == wJ ? at_J : tiles_of(w);
        if (w == wJ) m &= ~1ull << (J & 63);
        if (w == (J + 1) >> 6) m &= ~(1ull << ((J + 1) & 63));
        return m;
      };
      // The own tile, for whose rows nothing has to be known first, the long-term tiles, the tile after.  (Errors of dK and dV 0.98 of
      // key_tile's; with the tile after in second place 1.003.  The own tile last: dV 0.82, but dK/dV 90.7 instead of 82.7 us at B=32 H=8
      // L=2000 d=8.)
      Word rest = rest_of(wJ);
      const int last = min(J + 1, NT - 1);
      auto next_of = [&](int w, Word m) __attribute__((always_inline)) -> int { return m ? 64 * w + __builtin_ctzll(m) : last; };
      Word m_lt[4], m_st[4];
      const bool diag = !kDiag && p.sblk == 1 && J + 2 < NT;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        m_lt[r] = own ? triangle(r, true) : 0ull;
        m_st[r] = nm.own[r];
      }
      tile(yes, yes, yes, J, diag ? J + 2 : next_of(wJ, rest), m_lt, m_st);
      if constexpr (!kDiag) {  // (per position: a single word)
        if (p.sblk == 1)
          for (int d = 2; J + d < NT; d *= 2) {
            const int t = J + d;
            const bool here = (rest >> (t & 63)) & 1ull;
            rest &= ~(1ull << (t & 63));
#pragma unroll
            for (int r = 0; r < 4; ++r) m_st[r] = triangle(r, false) & triangle(r, true);
            const int t_next = J + 2 * d < NT ? J + 2 * d : next_of(wJ, rest);
            if (here) tile(yes, yes, no, t, t_next, m_lt, m_st);
            else tile(no, yes, no, t, t_next, m_lt, m_st);
          }
      }
      for (int w = wJ;;) {
        while (rest) {
          const int t = 64 * w + __builtin_ctzll(rest);
          rest &= rest - 1;
          tile(yes, no, no, t, next_of(w, rest), m_lt, m_st);
        }
        if (ONE_WORD || ++w > wE) break;
        rest = rest_of(w);
        request(next_of(w, rest));
      }
      if (J + 1 == NT) return;
      if (after) tile(yes, yes, no, J + 1, J, m_lt, nm.next);
      else tile(no, yes, no, J + 1, J, m_lt, nm.next);
    };
    auto far_queries = [&]() __attribute__((always_inline)) {
      float kd[CPL], vd[CPL];
      Ops::floats(kf, kd);
      Ops::floats(vf, vd);
      float kw[CPL * 4], vw[CPL * 4];
      if constexpr (D == 8) {
        whole_row(kd, kw);
        whole_row(vd, vw);
      }
      diagonals(p, J, J, NT - 1, [&](int d) __attribute__((always_inline)) {
        // this lane group's distance
        const int i = j + kTile * d * (1 << g), tg = min(J + d * (1 << g), NT - 1);
        auto constant = [&](int k) { return src.row_constant(hl, tg, k); };
        const bool ok = i < p.L;
        if constexpr (D == 8) {
          float qr[D], gr[D];
          Qr.whole(tg, qr);
          Gr.whole(tg, gr);
          const float e = __builtin_amdgcn_exp2f(arg(dot_n(kw, qr, 0.0f), constant(5)));
          const float pr = ok ? e : 0.0f, zd = constant(1), as = 1.0f - constant(0);
          t_st = fmaf(zd, pr, t_st);
          add_row(dv_part, as * pr, gr);
          add_row(dk_part, pr * fmaf(as, dot_n(vw, gr, 0.0f), fmaf(zd, wv_st, -constant(3))), qr);
        } else {
          float s[4], x[4], qo[4][NMB][4], go[4][NMB][4];
#pragma unroll
          for (int n = 0; n < 4; ++n) {
            float qr[CPL], gr[CPL];
            const int t = min(J + d * (1 << n), NT - 1);
            Qr.row(t, qr);
            Gr.row(t, gr);
            s[n] = dot_n(kd, qr, 0.0f);
            x[n] = dot_n(vd, gr, 0.0f);
            if constexpr (D == 16) {
              own_of_row(qr, qo[n]);
              own_of_row(gr, go[n]);
            }
          }
          phase_end<D>();
          if constexpr (D != 16) {
#pragma unroll
            for (int n = 0; n < 4; ++n) {
              const int t = min(J + d * (1 << n), NT - 1);
              Qr.own(t, qo[n]);
              Gr.own(t, go[n]);
            }
          }
          const float e = __builtin_amdgcn_exp2f(arg(gather_g(s), constant(5))), gd = gather_g(x);
          const float pr = ok ? e : 0.0f;
          const float zd = constant(1), as = 1.0f - constant(0);
          t_st = fmaf(zd, pr, t_st);
          spread_g(as * pr, s);
          spread_g(pr * fmaf(as, gd, fmaf(zd, wv_st, -constant(3))), x);
          add_own(dv_part, s, go);
          add_own(dk_part, x, qo);
        }
      });
    };
    if (kDiag && kFarFirst<D> && p.sblk == 1) far_queries();
    walk();
    if (kDiag && !kFarFirst<D> && p.sblk == 1) far_queries();
    // the gate part of dV: sum_i dz_i P_ij times the gate row of the branch
    if constexpr (Geo<D>::kQuads) {  // (a lane's part of the sums, like the accumulators)
#pragma unroll
      for (int h = 0; h < NACC; ++h) {
        float x[4], y[4];
        load_n<4>(wrow + 4 * h, x);
        load_n<4>(wrow + D + 4 * h, y);
#pragma unroll
        for (int r = 0; r < 4; ++r) dv_part[h][r] += fmaf(t_lt, x[r], t_st * y[r]);
      }
    } else {
      t_lt = sum_g(t_lt);
      t_st = sum_g(t_st);
#pragma unroll
      for (int mb = 0; mb < NMB; ++mb) {
        float x[4], y[4];
        load_n<4>(wrow + 16 * mb + 4 * g, x);
        load_n<4>(wrow + D + 16 * mb + 4 * g, y);
#pragma unroll
        for (int r = 0; r < 4; ++r) dv_part[mb][r] += fmaf(t_lt, x[r], t_st * y[r]);
      }
    }
  }
  f32x4 dk[NMB], dv[NMB];
  total<D>(dk_part, dk);
  total<D>(dv_part, dv);
  if constexpr (kEarly) arrived();
  else more();
  const int el = fresh_lane(), ej = J * kTile + (el & 15);
  if (ej < p.L) {
    store_grad_row<T, D>(dK_head + (unsigned)ej * D, dk, p.scale, ej >= p0, p, true, ej, el >> 4);
    store_grad_row<T, D>(dV_head + (unsigned)ej * D, dv, 1.0f, ej >= p0, p, false, ej, el >> 4);
  }
  return __ballot(!((ej < p0) | (ej >= p.L) | finite(abs_sum(dk) + abs_sum(dv)))) == 0ull;
}

// A wavefront's part of LDS where streamed tiles are turned: `tensors` tiles of rows, read back by columns (an operand by columns is
// four loads and more of one element a lane, sixteen vector-memory instructions a tile in dK/dV, whose address unit they filled), and
// the tile's row constants.
constexpr int kStreamWaves = 4;
template <typename T, int D>
constexpr int turn_floats(int tensors)
{
  return tensors * kTile * kLdsRow<T, D> + 6 * kTile;
}
// the n-th tile of a wavefront of W: there and back, so that the shorter walks of a round meet the longer ones of the next
__device__ __forceinline__ int to_and_fro(int n, int wv, int W) { return n * W + ((n & 1) ? W - 1 - wv : wv); }

}  // namespace

// =============================================================================================
// backward, heads streamed from memory: gate pass and dQ, then dK/dV
// =============================================================================================
// What the dK/dV kernel reads (SmallWs): per query tile the row constants [6][16] (alpha, dz, D_lt, D_st and the two lse
// in log2 units; rows that take no part have lse 1e30: every probability zero), its long-term tile words [NWt], and the
// selection bits per query block (block size 8) or per position.
// stages: kBwdStageGate writes those and the partial gate gradients, kBwdStageDQ writes dQ (the row constants are
// formed in either case).
// (Wavefronts per SIMD, here and in the dK/dV kernel: those that the walk's registers allow, which the compiler would exceed for
// the repeated walk.  d = 8 at B=32 H=8 L=2000: dQ with six 78 us, with five 69.)
template <typename T, int D, int BK, bool PERPOS>
__global__ __launch_bounds__(64 * kMaxWaves) __attribute__((amdgpu_waves_per_eu(D == 32 ? 4 : 5))) void bwd_dq_small_kernel(
    const T *__restrict__ Q, const T *__restrict__ K, const T *__restrict__ V, const int *__restrict__ valid_len,
    const int *__restrict__ sel, const float *__restrict__ gate_w, const float *__restrict__ gate_b,
    const float *__restrict__ o_lt, const float *__restrict__ o_st, const float *__restrict__ lse_lt,
    const float *__restrict__ lse_st, const T *__restrict__ dO, T *__restrict__ dQ, SmallWs ws, int hpg, int parts,
    unsigned stages, KParams p)
{
  constexpr int GW = 2 * D + 1;
  extern __shared__ __attribute__((aligned(16))) float small_lds[];  // the wavefronts' selection words
  __shared__ float red[kMaxWaves][GW];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), W = blockDim.x >> 6;
  const unsigned vid = mfma::xcd_spread(blockIdx.x, gridDim.x / parts, parts);
  const int bh = (int)(vid / parts), part = (int)(vid % parts);
  const int NT = (p.L + kTile - 1) / kTile, NWt = (NT + 31) / 32;
  const int p0 = p.L - clamp_len(valid_len[bh / p.H], p.L);
  const int T0 = p0 / kTile;
  const int q = lane & 15, g = lane >> 4;
  const int kvh = PERPOS ? bh / hpg : bh;
  const Rows<T, D> Kr(K + (size_t)kvh * p.L * D, p.L, q, g), Vr(V + (size_t)kvh * p.L * D, p.L, q, g);
  const QueryHead in(Q, dO, o_lt, o_st, lse_lt, lse_st, bh, p.L, D);
  GateSums<D> gate(gate_w, gate_b, bh % p.H);
  unsigned *my_lds = reinterpret_cast<unsigned *>(small_lds) + wv * lt_words(p, PERPOS);
  T *dQ_head = dQ + (size_t)bh * p.L * D;
  const LaneMasks lm = LaneMasks::make(p, q, g);
  const bool do_rows = stages & kBwdStageGate, do_dq = stages & kBwdStageDQ;
  auto sink = [&](int I, float al, float dz, float D_lt, float D_st, float l2_lt, float l2_st, const LtSel<BK, PERPOS> &ls, const auto &,
                  const auto &) __attribute__((always_inline)) {
    const int el = fresh_lane(), eq = el & 15, eg = el >> 4;
    float *rc = ws.rowc + ((size_t)bh * NT + I) * (6 * kTile);
    // lane group 0 writes alpha, group 1 dz, 2 D_lt, 3 D_st; groups 0 and 1 then the two lse
    rc[el] = eg == 0 ? al : eg == 1 ? dz : eg == 2 ? D_lt : D_st;
    if (eg < 2) rc[64 + el] = eg == 0 ? l2_lt : l2_st;
    if (PERPOS && bh % hpg != 0) return;
    for (int i = el; i < NWt; i += 64) ws.tile_words[((size_t)kvh * NT + I) * NWt + i] = ls.tiles[i];
    if constexpr (PERPOS) {
      if (eg == 0) store_pair(ws.sel_bits + ((size_t)kvh * NT * kTile + I * kTile + eq) * 2, ls.row);
    } else if constexpr (BK < kTile) {
      for (int i = el; i < 2 * ls.NWb; i += 64) ws.sel_bits[((size_t)kvh * NT + I) * 2 * ls.NWb + i] = ls.bits[i];
    }
  };
  const int *sel_head = sel + (size_t)kvh * (PERPOS ? p.L : p.NB) * p.k;
  bool good = true;
  for (int u = part * W + wv; u < NT; u += parts * W) {
    const int I = NT - 1 - u;
    if (I < T0 || p0 >= p.L) {  // no valid query
      if (do_dq) zero_fill(dQ_head + I * kTile * D, min(kTile, p.L - I * kTile) * D, fresh_lane());
      continue;
    }
    good &= query_tile<T, D, BK, PERPOS, false>(p, I, T0, NT, p0, lane, in, Kr, Vr, sel_head, my_lds, gate, lm, do_rows, do_dq, dQ_head, sink);
  }
  if (do_rows) gate.finish(red, ws.partial + ((size_t)bh * parts + part) * GW, lane, wv, W);
  if (__builtin_expect(!good, 0))
    query_tiles_carefully<T, D, BK, PERPOS>(p, part * W + wv, parts * W, T0, NT, p0, lane, in, Kr, Vr, sel_head, my_lds, gate_w, gate_b,
                                            bh % p.H, dQ_head);
}

template <typename T, int D, int BK, bool PERPOS>
__global__ __launch_bounds__(64 * kMaxWaves) __attribute__((amdgpu_waves_per_eu(D == 32 ? 3 : 4))) void bwd_dkv_small_kernel(
    const T *__restrict__ Q, const T *__restrict__ K, const T *__restrict__ V, const int *__restrict__ valid_len,
    const float *__restrict__ gate_w, const T *__restrict__ dO, SmallWs ws, T *__restrict__ dK, T *__restrict__ dV, int hpg, int parts,
    KParams p)
{
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), W = blockDim.x >> 6;
  const unsigned vid = mfma::xcd_spread(blockIdx.x, gridDim.x / parts, parts);
  const int bg = (int)(vid / parts), part = (int)(vid % parts);
  const int NT = (p.L + kTile - 1) / kTile, NWt = (NT + 31) / 32, NWb = (p.NB + 31) / 32;
  const int p0 = p.L - clamp_len(valid_len[bg / (p.H / hpg)], p.L);
  const int T0 = p0 / kTile;
  const int q = lane & 15, g = lane >> 4;
  const size_t head_kv = (size_t)bg * p.L * D;
  const Rows<T, D> Kr(K + head_kv, p.L, q, g), Vr(V + head_kv, p.L, q, g);
  struct {
    const T *Q, *dO;
    const float *rowc, *gate_w;
    const unsigned *bits;
    Slice words;
    int bh0, H, L, NT, NWt, q, g;
    __device__ __forceinline__ Rows<T, D> q_rows(int hl) const { return Rows<T, D>(Q + (size_t)(bh0 + hl) * L * D, L, q, g); }
    __device__ __forceinline__ Rows<T, D> g_rows(int hl) const { return Rows<T, D>(dO + (size_t)(bh0 + hl) * L * D, L, q, g); }
    __device__ __forceinline__ const float *gate_row(int hl) const { return gate_w + (size_t)((bh0 + hl) % H) * 2 * D; }
    __device__ __forceinline__ void constant(int hl, int I, int k, float (&x)[4]) const
    {
      const Slice rc(rowc + (size_t)(bh0 + hl) * NT * (6 * kTile), (size_t)NT * (6 * kTile) * 4);
      load_n<float>(rc, (unsigned)(I * (6 * kTile) + 16 * k + 4 * g) * 4u, x);
    }
    __device__ __forceinline__ float row_constant(int hl, int I, int k) const  // of row q of tile I
    {
      const Slice rc(rowc + (size_t)(bh0 + hl) * NT * (6 * kTile), (size_t)NT * (6 * kTile) * 4);
      return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rc.d, (unsigned)(I * (6 * kTile) + 16 * k + q) * 4u, 0, 0));
    }
    __device__ __forceinline__ unsigned tile_word(int I, int w) const
    {
      return __builtin_amdgcn_raw_buffer_load_b32(words.d, 4u * (unsigned)(I * NWt + w), 0, 0);
    }
  } src = {Q, dO, ws.rowc, gate_w, ws.sel_bits + (size_t)bg * (PERPOS ? NT * kTile * 2 : NT * 2 * NWb),
           Slice(ws.tile_words + (size_t)bg * NT * NWt, (size_t)NT * NWt * 4), bg * hpg, p.H, p.L, NT, NWt, q, g};
  bool good = true;
  for (int J = part * W + wv; J < NT; J += parts * W) {
    if (J < T0 || p0 >= p.L) {  // no valid key
      const int cnt = min(kTile, p.L - J * kTile) * D, el = fresh_lane();
      zero_fill(dK + head_kv + (size_t)J * kTile * D, cnt, el);
      zero_fill(dV + head_kv + (size_t)J * kTile * D, cnt, el);
      continue;
    }
    typename Operands<T, D>::Row kf, vf;
    Kr.op(J, kf);
    Vr.op(J, vf);
    good &= key_tile<T, D, BK, PERPOS, false>(p, J, T0, NT, p0, lane, kf, vf, hpg, src, dK + head_kv, dV + head_kv);
  }
  if (__builtin_expect(!good, 0))
    for (int J = part * W + wv; J < NT; J += parts * W) {
      if (J < T0) continue;
      typename Operands<T, D>::Row kf, vf;
      Kr.op(J, kf);
      Vr.op(J, vf);
      key_tile<T, D, BK, PERPOS, true>(p, J, T0, NT, p0, lane, kf, vf, hpg, src, dK + head_kv, dV + head_kv);
    }
}

// =============================================================================================
// backward, whole heads in LDS: gate pass, dQ and dK/dV of a (row, head), or of a (row, group), in one workgroup
// =============================================================================================
// K and V are staged, the query tiles run (each leaving its Q and dO rows, row constants and selection in LDS), then the key
// tiles.  Every tensor comes from memory once, in two round trips.  overlay: Q and dO do not fit beside K and V; they take
// their place after the query tiles, read a second time (from L2).
// ORDER: see HEADS BY LENGTH (a kernel of its own: beside it, though never taken, the code cost B=2048 H=8 L=200 1-2 %).
template <typename T, int D, int BK, bool PERPOS, bool ORDER>
__global__ __launch_bounds__(64 * kMaxWaves) __attribute__((amdgpu_waves_per_eu(4))) void bwd_res_kernel(
    const T *__restrict__ Q, const T *__restrict__ K, const T *__restrict__ V, const int *__restrict__ valid_len,
    const int *__restrict__ sel, const float *__restrict__ gate_w, const float *__restrict__ gate_b,
    const float *__restrict__ o_lt, const float *__restrict__ o_st, const float *__restrict__ lse_lt,
    const float *__restrict__ lse_st, const T *__restrict__ dO, T *__restrict__ dQ, T *__restrict__ dK, T *__restrict__ dV,
    float *__restrict__ partial, int hpg, int overlay, unsigned stages, KParams p)
{
  constexpr int GW = 2 * D + 1;
  extern __shared__ __attribute__((aligned(16))) float small_lds[];
  __shared__ float red[kMaxWaves][GW];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), W = blockDim.x >> 6;
  // (row, key/value head)
  const Unit unit = [&]() -> Unit {
    if constexpr (ORDER) return place_by_length(valid_len, p, p.H / hpg, wv);
    else return {(int)blockIdx.x, clamp_len(valid_len[blockIdx.x / (p.H / hpg)], p.L)};
  }();
  const int bg = unit.id;
  const int NT = (p.L + kTile - 1) / kTile, NWt = (NT + 31) / 32, NWb = (p.NB + 31) / 32;
  const int p0 = p.L - unit.valid;
  const int T0 = p0 / kTile;
  const int q = lane & 15, g = lane >> 4;
  const size_t head_kv = (size_t)bg * p.L * D;
  const bool do_dq = stages & kBwdStageDQ, do_dkv = stages & kBwdStageDKV;  // (the gate pass belongs to the query tiles)
  const ResLayout lay(p, kLdsRow<T, D>, PERPOS, hpg, overlay, W);
  float *Ks = small_lds, *Vs = Ks + lay.pitch, *QG = small_lds + lay.qg, *rc = small_lds + lay.rowc;
  unsigned *words = reinterpret_cast<unsigned *>(small_lds + lay.words), *bits = words + NT * NWt;
  unsigned *my_lds = reinterpret_cast<unsigned *>(small_lds + lay.waves) + wv * lt_words(p, PERPOS);

  // CLEAN: a row that sees a key or a value that is not finite has saved outputs that are not, and takes its NaN from there
  stage_pair<T, D, true>(K + head_kv, V + head_kv, Ks, Vs, p.L, T0, NT, p0, lane, wv, W);
  __syncthreads();
  const LdsRows<T, D> Kr(Ks, q, g), Vr(Vs, q, g);
  const LaneMasks lm = LaneMasks::make(p, q, g);
  const int *sel_head = sel + (size_t)bg * (PERPOS ? p.L : p.NB) * p.k;
  for (int hl = 0; hl < hpg; ++hl) {
    const int bh = bg * hpg + hl;
    const QueryHead in(Q, dO, o_lt, o_st, lse_lt, lse_st, bh, p.L, D);
    GateSums<D> gate(gate_w, gate_b, bh % p.H);
    T *dQ_head = dQ + (size_t)bh * p.L * D;
    auto sink = [&](int I, float al, float dz, float D_lt, float D_st, float l2_lt, float l2_st, const LtSel<BK, PERPOS> &ls,
                    const typename Operands<T, D>::Row &q_op, const typename Operands<T, D>::Row &g_op) __attribute__((always_inline)) {
      float *c = rc + (hl * NT + I) * (6 * kTile);
      c[lane] = g == 0 ? al : g == 1 ? dz : g == 2 ? D_lt : D_st;
      if (g < 2) c[64 + lane] = g == 0 ? l2_lt : l2_st;
      if (!overlay) {
        LdsRows<T, D>::put(QG + 2 * hl * lay.pitch, I * kTile + q, g, q_op);
        LdsRows<T, D>::put(QG + (2 * hl + 1) * lay.pitch, I * kTile + q, g, g_op);
      }
      if (hl > 0) return;
      for (int i = lane; i < NWt; i += 64) words[I * NWt + i] = ls.tiles[i];
      if constexpr (PERPOS) {
        if (g == 0) store_pair(bits + (I * kTile + q) * 2, ls.row);
      } else if constexpr (BK < kTile) {
        for (int i = lane; i < 2 * NWb; i += 64) bits[I * 2 * NWb + i] = ls.bits[i];
      }
    };
    for (int u = wv; u < NT; u += W) {
      const int I = NT - 1 - u;
      if (I < T0 || p0 >= p.L) {  // no valid query
        if (do_dq) zero_fill(dQ_head + I * kTile * D, min(kTile, p.L - I * kTile) * D, fresh_lane());
        continue;
      }
      query_tile<T, D, BK, PERPOS, false>(p, I, T0, NT, p0, lane, in, Kr, Vr, sel_head, my_lds, gate, lm, true, do_dq, dQ_head, sink);
    }
    if (hl > 0) __syncthreads();
    gate.finish(red, partial + (size_t)bh * GW, lane, wv, W);  // (its barrier also closes the query tiles of the head)
  }
  if (!do_dkv) return;
  typename Operands<T, D>::Row kf, vf;
  if (overlay) {
    __syncthreads();
    for (int hl = 0; hl < hpg; ++hl) {
      const size_t at = (size_t)(bg * hpg + hl) * p.L * D;
      stage_pair<T, D, false>(Q + at, dO + at, QG + 2 * hl * lay.pitch, QG + (2 * hl + 1) * lay.pitch, p.L, T0, NT, p0, lane, wv, W);
    }
    __syncthreads();
  }
  struct {
    const float *qg, *rc, *gate_w;
    const unsigned *bits, *words;
    int bh0, H, NT, NWt, q, g, pitch;
    __device__ __forceinline__ LdsRows<T, D> q_rows(int hl) const { return LdsRows<T, D>(qg + 2 * hl * pitch, q, g); }
    __device__ __forceinline__ LdsRows<T, D> g_rows(int hl) const { return LdsRows<T, D>(qg + (2 * hl + 1) * pitch, q, g); }
    __device__ __forceinline__ const float *gate_row(int hl) const { return gate_w + (size_t)((bh0 + hl) % H) * 2 * D; }
    __device__ __forceinline__ void constant(int hl, int I, int k, float (&x)[4]) const
    {
      load_n<4>(rc + (hl * NT + I) * (6 * kTile) + 16 * k + 4 * g, x);
    }
    __device__ __forceinline__ float row_constant(int hl, int I, int k) const { return rc[(hl * NT + I) * (6 * kTile) + 16 * k + q]; }
    __device__ __forceinline__ unsigned tile_word(int I, int w) const { return words[I * NWt + w]; }
  } src = {QG, rc, gate_w, bits, words, bg * hpg, p.H, NT, NWt, q, g, lay.pitch};
  const Rows<T, D> Kg(K + head_kv, p.L, q, g), Vg(V + head_kv, p.L, q, g);
  bool good = true;
  for (int u = wv; u < NT; u += W) {
    const int J = (T0 + u) % NT;  // the tiles without a valid key come last
    if (J < T0 || p0 >= p.L) {
      const int cnt = min(kTile, p.L - J * kTile) * D, el = fresh_lane();
      zero_fill(dK + head_kv + (size_t)J * kTile * D, cnt, el);
      zero_fill(dV + head_kv + (size_t)J * kTile * D, cnt, el);
      continue;
    }
    if (overlay) {
      Kg.op(J, kf);
      Vg.op(J, vf);
    } else {
      Kr.op(J, kf);
      Vr.op(J, vf);
    }
    good &= key_tile<T, D, BK, PERPOS, false>(p, J, T0, NT, p0, lane, kf, vf, hpg, src, dK + head_kv, dV + head_kv);
  }
  if (__builtin_expect(!good, 0))
    for (int u = wv; u < NT - T0; u += W) {
      Kg.op(T0 + u, kf);
      Vg.op(T0 + u, vf);
      key_tile<T, D, BK, PERPOS, true>(p, T0 + u, T0, NT, p0, lane, kf, vf, hpg, src, dK + head_kv, dV + head_kv);
    }
}

// =============================================================================================
// backward, whole heads in LDS, THE NEAR FORM
// =============================================================================================
// As bwd_res_kernel, and as in fwd_near_kernel: what the next tile needs is on its way during the walk and has arrived before the stores
// go out, masks are scalars, the selection stays in registers.  The (tile, head) pairs of a group are dealt out over all of its heads
// without a barrier between them, there and back; Q and dO are requested before the barrier that closes K and V; the gate row lies
// in LDS.  us, with bwd_res_kernel / with this: B=2048 H=8 L=200 d=16 603 / 550 (vector instructions 1390 a pair of tiles before),
// per position at d=8 560 / 502, B=256 H=2 L=200 d=32 43.8 / 39.4.
template <typename T, int D, int BK, bool PERPOS, bool ORDER>
__global__ __launch_bounds__(64 * kMaxWaves) __attribute__((amdgpu_waves_per_eu(4))) void bwd_near_kernel(
    const T *__restrict__ Q, const T *__restrict__ K, const T *__restrict__ V, const int *__restrict__ valid_len,
    const int *__restrict__ sel, const float *__restrict__ gate_w, const float *__restrict__ gate_b,
    const float *__restrict__ o_lt, const float *__restrict__ o_st, const float *__restrict__ lse_lt,
    const float *__restrict__ lse_st, const T *__restrict__ dO, T *__restrict__ dQ, T *__restrict__ dK, T *__restrict__ dV,
    float *__restrict__ partial, int hpg, int overlay, unsigned stages, NearMasks nm_q, NearMasks nm_k, KParams p)
{
  constexpr int GW = 2 * D + 1;
  using Ops = Operands<T, D>;
  extern __shared__ __attribute__((aligned(16))) float small_lds[];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), W = blockDim.x >> 6;
  if constexpr (!PERPOS) hpg = 1;
  // (row, key/value head)
  const Unit unit = [&]() -> Unit {
    if constexpr (ORDER) return place_by_length(valid_len, p, p.H / hpg, wv);
    else return {(int)blockIdx.x, clamp_len(valid_len[blockIdx.x / (p.H / hpg)], p.L)};
  }();
  const int bg = unit.id;
  const int NT = (p.L + kTile - 1) / kTile, NWt = (NT + 31) / 32, NWb = (p.NB + 31) / 32;
  const int p0 = p.L - unit.valid;
  const int T0 = p0 / kTile;
  const int q = lane & 15, g = lane >> 4;
  const size_t head_kv = (size_t)bg * p.L * D;
  const bool do_dq = stages & kBwdStageDQ, do_dkv = stages & kBwdStageDKV;  // (the gate pass belongs to the query tiles)
  const ResLayout lay(p, kLdsRow<T, D>, PERPOS, hpg, overlay, W);
  float *Ks = small_lds, *Vs = Ks + lay.pitch, *QG = small_lds + lay.qg, *rc = small_lds + lay.rowc;
  float *gates = small_lds + lay.gates, *red = small_lds + lay.red;
  unsigned *words = reinterpret_cast<unsigned *>(small_lds + lay.words), *bits = words + NT * NWt;
  unsigned *my_lds = reinterpret_cast<unsigned *>(small_lds + lay.waves) + wv * lt_words(p, PERPOS);
  const int bh0 = bg * hpg, h0 = bh0 % p.H;
  const int count = p0 >= p.L ? 0 : NT - T0;  // tiles with a valid position

  // ---- query tiles: pair (tile, head) number x is tile NT - 1 - x % count of head x / count ----
  const int *sel_head = sel + (size_t)bg * (PERPOS ? p.L : p.NB) * p.k;
  auto head = [&](int hl) { return QueryHead(Q, dO, o_lt, o_st, lse_lt, lse_st, bh0 + hl, p.L, D); };
  const int pairs = count * hpg;
  int n = 0, x = wv, hl = 0, at = wv;  // this wavefront's next pair: number, head, place in the head
  while (at >= count && hl < hpg - 1) at -= count, ++hl;
  QueryIn<T, D, BK, PERPOS> in;
  in.request(p, NT - 1 - at, p0, lane, head(hl), sel_head, x < pairs);
  for (int i = threadIdx.x; i < hpg * 2 * D; i += blockDim.x) gates[i] = gate_w[(size_t)h0 * 2 * D + i];
  if constexpr (NearGateSums<D>::kInLds)
    for (int i = threadIdx.x; i < hpg * W * GW; i += blockDim.x) red[i] = 0.0f;
  // CLEAN: a row that sees a key or a value that is not finite has saved outputs that are not, and takes its NaN from there
  stage_pair<T, D, true, kStageAhead<D>>(K + head_kv, V + head_kv, Ks, Vs, p.L, T0, NT, p0, lane, wv, W);
  __syncthreads();
  const LdsRows<T, D> Kr(Ks, q, g), Vr(Vs, q, g);
  Word valid_keys[4];  // of the first tile
#pragma unroll
  for (int r = 0; r < 4; ++r) valid_keys[r] = elements_from(p0 & (kTile - 1), r);
  for (int hh = 0; hh < hpg; ++hh) {
    NearGateSums<D> gate(gate_b, h0 + hh, red + (hh * W + wv) * GW);
    T *dQ_head = dQ + (size_t)(bh0 + hh) * p.L * D;
    auto sink = [&](int I, float al, float dz, float D_lt, float D_st, float l2_lt, float l2_st, const LtSel<BK, PERPOS> &ls,
                    const typename Ops::Row &q_op, const typename Ops::Row &g_op, auto &&tiles_of) __attribute__((always_inline)) {
      float *c = rc + (hh * NT + I) * (6 * kTile);
      c[lane] = g == 0 ? al : g == 1 ? dz : g == 2 ? D_lt : D_st;
      if (g < 2) c[64 + lane] = g == 0 ? l2_lt : l2_st;
      if (!overlay) {
        LdsRows<T, D>::put(QG + 2 * hh * lay.pitch, I * kTile + q, g, q_op);
        LdsRows<T, D>::put(QG + (2 * hh + 1) * lay.pitch, I * kTile + q, g, g_op);
      }
      if (hh > 0) return;
      const Word all = tiles_of(0);
      if (lane < NWt) words[I * NWt + lane] = lane == 0 ? (unsigned)all : (unsigned)(all >> 32);
      if constexpr (PERPOS) {
        if (g == 0) store_pair(bits + (I * kTile + q) * 2, ls.row);
      } else if constexpr (BK < kTile) {
        for (int i = lane; i < 2 * NWb; i += 64) bits[I * 2 * NWb + i] = ls.bits[i];
      }
    };
    while (x < pairs && hl <= hh) {
      const int I = NT - 1 - at;
      ++n;
      const int x_next = to_and_fro(n, wv, W);
      at += x_next - x;
      x = x_next;
      while (at >= count && hl < hpg) at -= count, ++hl;
      near_query_tile<T, D, BK, PERPOS, true>(
          p, I, T0, NT, p0, lane, in, Kr, Vr, sel_head, my_lds, gates + hh * 2 * D, gate, nm_q, valid_keys, true, do_dq, dQ_head,
          [&](QueryIn<T, D, BK, PERPOS> &next) __attribute__((always_inline)) {
            next.request(p, NT - 1 - at, p0, lane, head(min(hl, hpg - 1)), sel_head, x < pairs);
          },
          sink);
    }
    gate.leave(lane);
  }

  // ---- between the two: Q and dO take the place of K and V (overlay), the gate sums are closed ----
  typename Ops::Row kf, vf, kn, vn;
  const Rows<T, D> Kg(K + head_kv, p.L, q, g), Vg(V + head_kv, p.L, q, g);
  auto fetch = [&](int u) __attribute__((always_inline)) {
    const unsigned off = u < count ? Kg.row_off + (unsigned)(T0 + u) * Rows<T, D>::TB : kNowhere;
    load_op<T, D>(Kg.s, off, kn);
    load_op<T, D>(Vg.s, off, vn);
    asm volatile("" ::: "memory");
  };
  if (do_dkv) fetch(wv);
  if (overlay && do_dkv) {
    for (int hh = 0; hh < hpg; ++hh) {
      const size_t from = (size_t)(bh0 + hh) * p.L * D;
      stage_pair<T, D, false, kStageAhead<D>>(Q + from, dO + from, QG + 2 * hh * lay.pitch, QG + (2 * hh + 1) * lay.pitch, p.L, T0, NT, p0, lane, wv, W,
                              [&] {
                                if (hh == 0) __syncthreads();
                              });
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < hpg * GW; i += blockDim.x) {
    const int hh = i / GW, c = i - hh * GW;
    float a = 0.0f;
    for (int w = 0; w < W; ++w) a += red[(hh * W + w) * GW + c];
    partial[(size_t)(bh0 + hh) * GW + c] = a;
  }
  bool good = true;
  if (do_dkv) {
    struct {
      const float *qg, *rc, *gates;
      const unsigned *bits, *words;
      int NT, NWt, q, g, pitch;
      __device__ __forceinline__ LdsRows<T, D> q_rows(int hl) const { return LdsRows<T, D>(qg + 2 * hl * pitch, q, g); }
      __device__ __forceinline__ LdsRows<T, D> g_rows(int hl) const { return LdsRows<T, D>(qg + (2 * hl + 1) * pitch, q, g); }
      __device__ __forceinline__ const float *gate_row(int hl) const { return gates + hl * 2 * D; }
      __device__ __forceinline__ void constant(int hl, int I, int k, float (&x)[4]) const
      {
        load_n<4>(rc + (hl * NT + I) * (6 * kTile) + 16 * k + 4 * g, x);
      }
      __device__ __forceinline__ float row_constant(int hl, int I, int k) const { return rc[(hl * NT + I) * (6 * kTile) + 16 * k + q]; }
      __device__ __forceinline__ unsigned tile_word(int I, int w) const { return words[I * NWt + w]; }
    } src = {QG, rc, gates, bits, words, NT, NWt, q, g, lay.pitch};
    for (int n = 0, u = wv; u < count;) {
      const int J = T0 + u;
      kf = kn;
      vf = vn;
      u = to_and_fro(++n, wv, W);
      good &= near_key_tile<T, D, BK, PERPOS, true>(
          p, J, T0, NT, p0, lane, kf, vf, hpg, src, nm_k, dK + head_kv, dV + head_kv, [&]() __attribute__((always_inline)) { fetch(u); },
          [&]() __attribute__((always_inline)) {
            Operands<T, D>::arrived(kn);
            Operands<T, D>::arrived(vn);
          });
    }
    if (__builtin_expect(!good, 0)) {
      struct {
        const float *qg, *rc, *gate_w;
        const unsigned *bits, *words;
        int NT, NWt, q, g, pitch;
        __device__ __forceinline__ LdsRows<T, D> q_rows(int hl) const { return LdsRows<T, D>(qg + 2 * hl * pitch, q, g); }
        __device__ __forceinline__ LdsRows<T, D> g_rows(int hl) const { return LdsRows<T, D>(qg + (2 * hl + 1) * pitch, q, g); }
        __device__ __forceinline__ const float *gate_row(int hl) const { return gate_w + (size_t)hl * 2 * D; }
        __device__ __forceinline__ void constant(int hl, int I, int k, float (&x)[4]) const
        {
          load_n<4>(rc + (hl * NT + I) * (6 * kTile) + 16 * k + 4 * g, x);
        }
        __device__ __forceinline__ float row_constant(int hl, int I, int k) const { return rc[(hl * NT + I) * (6 * kTile) + 16 * k + q]; }
        __device__ __forceinline__ unsigned tile_word(int I, int w) const { return words[I * NWt + w]; }
      } again = {QG, rc, gate_w + (size_t)h0 * 2 * D, bits, words, NT, NWt, q, g, lay.pitch};
      for (int n = 0, u = wv; u < count; u = to_and_fro(++n, wv, W)) {
        Kg.op(T0 + u, kf);
        Vg.op(T0 + u, vf);
        key_tile<T, D, BK, PERPOS, true>(p, T0 + u, T0, NT, p0, lane, kf, vf, hpg, again, dK + head_kv, dV + head_kv);
      }
    }
  }
  // ---- positions before the first tile with a valid one: zeros ----
  const int rows = min((NT - count) * kTile, p.L);
  for (int hh = 0; hh < hpg; ++hh)
    if (do_dq) zero_rows_from(dQ + (size_t)(bh0 + hh) * p.L * D, rows * D, (int)threadIdx.x, (int)blockDim.x);
  if (do_dkv) {
    zero_rows_from(dK + head_kv, rows * D, (int)threadIdx.x, (int)blockDim.x);
    zero_rows_from(dV + head_kv, rows * D, (int)threadIdx.x, (int)blockDim.x);
  }
}

// =============================================================================================
// backward, heads streamed from memory, THE NEAR FORM
// =============================================================================================
// As bwd_dq_small_kernel and bwd_dkv_small_kernel, and as bwd_near_kernel.  Tiles are turned in LDS (turn_floats): dK/dV issued sixteen
// vector-memory instructions a tile and waited for the address unit, five now.  us, with those / with these, B=32 H=8 L=2000 d=8: dQ 69 / 63, dK/dV
// 101 / 82; a whole step 241 / 200.  (The forward's values turned the same way: 53.3 / 52.5 and, at
// d=16, slower: its five instructions a tile stay.)
template <typename T, int D, int BK, bool PERPOS>
__global__ __launch_bounds__(64 * kMaxWaves) __attribute__((amdgpu_waves_per_eu(D == 8 ? 5 : 4))) void bwd_dq_near_kernel(
    const T *__restrict__ Q, const T *__restrict__ K, const T *__restrict__ V, const int *__restrict__ valid_len,
    const int *__restrict__ sel, const float *__restrict__ gate_w, const float *__restrict__ gate_b,
    const float *__restrict__ o_lt, const float *__restrict__ o_st, const float *__restrict__ lse_lt,
    const float *__restrict__ lse_st, const T *__restrict__ dO, T *__restrict__ dQ, SmallWs ws, int hpg, int parts,
    unsigned stages, NearMasks nm, KParams p)
{
  constexpr int GW = 2 * D + 1;
  extern __shared__ __attribute__((aligned(16))) float small_lds[];  // the wavefronts' selection words
  __shared__ __attribute__((aligned(16))) float gate_s[2 * D];
  __shared__ float red[kStreamWaves][GW];
  __shared__ __attribute__((aligned(16))) float turn_s[kStreamWaves][turn_floats<T, D>(1)];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), W = blockDim.x >> 6;
  const unsigned vid = mfma::xcd_spread(blockIdx.x, gridDim.x / parts, parts);
  const int bh = (int)(vid / parts), part = (int)(vid % parts);
  const int b = bh / p.H, h = bh - b * p.H;
  const int NT = (p.L + kTile - 1) / kTile, NWt = (NT + 31) / 32;
  const int p0 = p.L - clamp_len(valid_len[b], p.L);
  const int T0 = p0 / kTile;
  const int I_first = p0 >= p.L ? NT : T0;
  const int q = lane & 15, g = lane >> 4;
  const int kvh = PERPOS ? bh / hpg : bh;
  const int *sel_head = sel + (size_t)kvh * (PERPOS ? p.L : p.NB) * p.k;
  const QueryHead head(Q, dO, o_lt, o_st, lse_lt, lse_st, bh, p.L, D);
  int I = NT - 1 - (part * W + wv);
  QueryIn<T, D, BK, PERPOS> in;
  in.request(p, I, p0, lane, head, sel_head, I >= I_first);
  for (int i = threadIdx.x; i < 2 * D; i += blockDim.x) gate_s[i] = gate_w[(size_t)h * 2 * D + i];
  const Rows<T, D> Kr(K + (size_t)kvh * p.L * D, p.L, q, g), Vr(V + (size_t)kvh * p.L * D, p.L, q, g);
  float *mine = red[wv];
  if (lane < GW) mine[lane] = 0.0f;
  if (lane + 64 < GW) mine[lane + 64] = 0.0f;
  NearGateSums<D> gate(gate_b, h, mine);
  unsigned *my_lds = reinterpret_cast<unsigned *>(small_lds) + wv * lt_words(p, PERPOS);
  T *dQ_head = dQ + (size_t)bh * p.L * D;
  const bool do_rows = stages & kBwdStageGate, do_dq = stages & kBwdStageDQ;
  Word valid_keys[4];  // of the first tile
#pragma unroll
  for (int r = 0; r < 4; ++r) valid_keys[r] = elements_from(p0 & (kTile - 1), r);
  auto sink = [&](int I, float al, float dz, float D_lt, float D_st, float l2_lt, float l2_st, const LtSel<BK, PERPOS> &ls, const auto &,
                  const auto &, auto &&tiles_of) __attribute__((always_inline)) {
    const int el = fresh_lane(), eq = el & 15, eg = el >> 4;
    float *rc = ws.rowc + ((size_t)bh * NT + I) * (6 * kTile);
    // lane group 0 writes alpha, group 1 dz, 2 D_lt, 3 D_st; groups 0 and 1 then the two lse
    rc[el] = eg == 0 ? al : eg == 1 ? dz : eg == 2 ? D_lt : D_st;
    if (eg < 2) rc[64 + el] = eg == 0 ? l2_lt : l2_st;
    if (PERPOS && bh % hpg != 0) return;
    unsigned *words = ws.tile_words + ((size_t)kvh * NT + I) * NWt;
    for (int w = 0; w <= I >> 6; ++w) {  // (no key tile after I asks)
      const Word m = tiles_of(w);
      if (el < min(2, NWt - 2 * w)) words[2 * w + el] = el == 0 ? (unsigned)m : (unsigned)(m >> 32);
    }
    if constexpr (PERPOS) {
      if (eg == 0) store_pair(ws.sel_bits + ((size_t)kvh * NT * kTile + I * kTile + eq) * 2, ls.row);
    } else if constexpr (BK < kTile) {
      for (int i = el; i < 2 * ls.NWb; i += 64) ws.sel_bits[((size_t)kvh * NT + I) * 2 * ls.NWb + i] = ls.bits[i];
    }
  };
  __syncthreads();
  bool good = true;
  while (I >= I_first) {
    const int now = I;
    I -= parts * W;
    good &= near_query_tile<T, D, BK, PERPOS, PERPOS>(
        p, now, T0, NT, p0, lane, in, Kr, Vr, sel_head, my_lds, gate_s, gate, nm, valid_keys, do_rows, do_dq, dQ_head,
        [&](QueryIn<T, D, BK, PERPOS> &next) __attribute__((always_inline)) { next.request(p, I, p0, lane, head, sel_head, I >= I_first); }, sink,
        turn_s[wv]);
  }
  if (do_rows) {
    gate.leave(lane);
    __syncthreads();
    for (int c = threadIdx.x; c < GW; c += blockDim.x) {
      float a = 0.0f;
      for (int w = 0; w < W; ++w) a += red[w][c];
      ws.partial[((size_t)bh * parts + part) * GW + c] = a;
    }
  }
  if (__builtin_expect(!good, 0))
    query_tiles_carefully<T, D, BK, PERPOS>(p, part * W + wv, parts * W, T0, NT, p0, lane, head, Kr, Vr, sel_head, my_lds, gate_w, gate_b, h,
                                            dQ_head);
  // positions before the first tile with a valid one: zeros
  if (do_dq)
    zero_rows_from(dQ_head, min(I_first * kTile, p.L) * D, part * (int)blockDim.x + (int)threadIdx.x, parts * (int)blockDim.x);
}

template <typename T, int D, int BK, bool PERPOS>
__global__ __launch_bounds__(64 * kMaxWaves) __attribute__((amdgpu_waves_per_eu(D == 32 ? 3 : 4))) void bwd_dkv_near_kernel(
    const T *__restrict__ Q, const T *__restrict__ K, const T *__restrict__ V, const int *__restrict__ valid_len,
    const float *__restrict__ gate_w, const T *__restrict__ dO, SmallWs ws, T *__restrict__ dK, T *__restrict__ dV, int hpg, int parts,
    NearMasks nm, KParams p)
{
  __shared__ __attribute__((aligned(16))) float turn_s[kStreamWaves][turn_floats<T, D>(2)];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), W = blockDim.x >> 6;
  const unsigned vid = mfma::xcd_spread(blockIdx.x, gridDim.x / parts, parts);
  const int bg = (int)(vid / parts), part = (int)(vid % parts);
  const int NT = (p.L + kTile - 1) / kTile, NWt = (NT + 31) / 32, NWb = (p.NB + 31) / 32;
  const int p0 = p.L - clamp_len(valid_len[bg / (p.H / hpg)], p.L);
  const int T0 = p0 / kTile;
  const int count = p0 >= p.L ? 0 : NT - T0;  // tiles with a valid position
  const int q = lane & 15, g = lane >> 4;
  const size_t head_kv = (size_t)bg * p.L * D;
  const Rows<T, D> Kr(K + head_kv, p.L, q, g), Vr(V + head_kv, p.L, q, g);
  typename Operands<T, D>::Row kf, vf, kn, vn;
  auto fetch = [&](int J) __attribute__((always_inline)) {
    const unsigned off = J < NT && count > 0 ? Kr.row_off + (unsigned)J * Rows<T, D>::TB : kNowhere;
    load_op<T, D>(Kr.s, off, kn);
    load_op<T, D>(Vr.s, off, vn);
    asm volatile("" ::: "memory");
  };
  // (the first tile of this wavefront's that is not before T0)
  const int first = part * W + wv, step = parts * W;
  const int J0 = first >= T0 ? first : first + (T0 - first + step - 1) / step * step;
  fetch(J0);
  struct {
    const T *Q, *dO;
    const float *rowc, *gate_w;
    const unsigned *bits;
    Slice words;
    int bh0, H, L, NT, NWt, q, g;
    __device__ __forceinline__ Rows<T, D> q_rows(int hl) const { return Rows<T, D>(Q + (size_t)(bh0 + hl) * L * D, L, q, g); }
    __device__ __forceinline__ Rows<T, D> g_rows(int hl) const { return Rows<T, D>(dO + (size_t)(bh0 + hl) * L * D, L, q, g); }
    __device__ __forceinline__ const float *gate_row(int hl) const { return gate_w + (size_t)((bh0 + hl) % H) * 2 * D; }
    __device__ __forceinline__ void constant(int hl, int I, int k, float (&x)[4]) const
    {
      const Slice rc(rowc + (size_t)(bh0 + hl) * NT * (6 * kTile), (size_t)NT * (6 * kTile) * 4);
      load_n<float>(rc, (unsigned)(I * (6 * kTile) + 16 * k + 4 * g) * 4u, x);
    }
    __device__ __forceinline__ void constants(int hl, int I, int lane, float (&x)[4]) const  // all of them, 16 bytes a lane
    {
      const Slice rc(rowc + (size_t)(bh0 + hl) * NT * (6 * kTile), (size_t)NT * (6 * kTile) * 4);
      load_n<float>(rc, lane < 24 ? (unsigned)(I * (6 * kTile) + 4 * lane) * 4u : kNowhere, x);
    }
    __device__ __forceinline__ float row_constant(int hl, int I, int k) const  // of row q of tile I
    {
      const Slice rc(rowc + (size_t)(bh0 + hl) * NT * (6 * kTile), (size_t)NT * (6 * kTile) * 4);
      return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rc.d, (unsigned)(I * (6 * kTile) + 16 * k + q) * 4u, 0, 0));
    }
    __device__ __forceinline__ unsigned tile_word(int I, int w) const
    {
      return __builtin_amdgcn_raw_buffer_load_b32(words.d, 4u * (unsigned)(I * NWt + w), 0, 0);
    }
  } src = {Q, dO, ws.rowc, gate_w, ws.sel_bits + (size_t)bg * (PERPOS ? NT * kTile * 2 : NT * 2 * NWb),
           Slice(ws.tile_words + (size_t)bg * NT * NWt, (size_t)NT * NWt * 4), bg * hpg, p.H, p.L, NT, NWt, q, g};
  bool good = true;
  if (count > 0)
    for (int J = J0; J < NT;) {
      const int now = J;
      kf = kn;
      vf = vn;
      J += step;
      good &= near_key_tile<T, D, BK, PERPOS, PERPOS>(
          p, now, T0, NT, p0, lane, kf, vf, hpg, src, nm, dK + head_kv, dV + head_kv, [&]() __attribute__((always_inline)) { fetch(J); },
          [&]() __attribute__((always_inline)) {
            Operands<T, D>::arrived(kn);
            Operands<T, D>::arrived(vn);
          },
          turn_s[wv]);
    }
  if (__builtin_expect(!good, 0))
    for (int J = J0; J < NT; J += step) {
      Kr.op(J, kf);
      Vr.op(J, vf);
      key_tile<T, D, BK, PERPOS, true>(p, J, T0, NT, p0, lane, kf, vf, hpg, src, dK + head_kv, dV + head_kv);
    }
  // positions before the first tile with a valid one: zeros
  const int rows = min((NT - count) * kTile, p.L);
  zero_rows_from(dK + head_kv, rows * D, part * (int)blockDim.x + (int)threadIdx.x, parts * (int)blockDim.x);
  zero_rows_from(dV + head_kv, rows * D, part * (int)blockDim.x + (int)threadIdx.x, parts * (int)blockDim.x);
}

// =============================================================================================
// launchers
// =============================================================================================
namespace {

bool small_shape(const KParams &p)
{
  return (p.d == 8 || p.d == 16 || p.d == 32) && (p.b == 8 || p.b == 16) && p.L <= 16384;
}

// How a launch is laid out: whether workgroups hold whole heads in LDS (then one workgroup per unit), wavefronts per workgroup,
// workgroups per unit.  units: query heads, or key/value heads where a workgroup serves a whole group.
struct SmallPlan {
  bool res, overlay;
  int waves, parts;
  size_t lds;
};
// LDS up to which a workgroup holds whole heads: two of them per CU at d = 32, three below, whose lighter walks want the wavefronts
// (a training step, us, by limit 76 / 50 / 40 KB: B=300 H=8 d=16 L=300 296 / 280 / 277, L=450 446 / 422 / 421, d=8 L=450 289 / 288 / 297,
// L=600 455 / 414 / 416; B=32 d=8 L=1000 110 / 98 / -; B=1024 H=2 d=32 L=200 339 / 410 / 411; in the near form 226 / 209 / 207, 348 / 336 /
// 336, 238 / 237 / 227, 339 / 287 / 287, 85 / 76 / 76, 231 / 300 / 299)
constexpr size_t kTwoPerCU = 76 * 1024;
size_t small_lds_limit(const KParams &p) { return p.d == 32 ? kTwoPerCU : 44 * 1024; }
// Few heads: eight wavefronts each, a head's latency counts.  Many: four, whose shares are longer and better balanced (always a
// multiple of the four SIMDs: with five or six wavefronts the backward took 1.4 times as long).  The near form's lighter walks are
// many earlier, from more than two heads to a CU on, the longer the head (at d = 32, where fewer fit a CU, short ones alone): a training
// step, fp32, lengths U[L/10,L], eight wavefronts / four, us:
//   heads               400                 600                1000                1600
//   d = 8          L=60   22.9 / 22.3   L=100  35.2 / 32.5  L=200  59.4 / 54.2  L=300 118.5 / 104.6
//                 L=150   31.1 / 34.8   L=300  55.9 / 62.5  L=300  78.8 / 76.9
//   d = 16        L=100   30.2 / 30.3   L=100  38.6 / 35.5  L=150  59.6 / 54.1  L=200 105.4 /  93.0
//                 L=200   38.7 / 44.5   L=200  53.1 / 52.9  L=200  70.7 / 64.9
//   d = 32         L=60   30.8 / 30.2    L=60  43.6 / 33.9   L=60  51.3 / 40.0   L=60  78.7 /  57.3
//                 L=200   58.4 / 67.0   L=100  54.3 / 57.7  L=200   107 /  115  L=200   165 /   176
//   per position  L=100   40.5 / 44.1   L=100  55.1 / 49.6  L=150  88.5 / 80.6  L=200   173 /   150
//                 L=200   62.8 / 80.5   L=150  61.3 / 65.0  L=200   111 /  107
bool many_heads(int units) { return units >= 2048; }
int res_waves(const KParams &p, int units, bool near)
{
  return many_heads(units) || (near && units > 2 * kCUs && (p.d == 32 ? p.L <= 64 : 5 * p.L <= units)) ? 4 : 8;
}
// More than one head to a CU (with one the order is of no account), and not so many that they average out.  The forward, a third of
// the backward's time, only where the order pays for itself: two heads to a CU of at least 128 positions (in the near form 150, or 112 at
// d = 32), or several query heads a workgroup (B=250 H=8 L=200 d=16 44.2 us in turn, 47.9 by length; B=128 H=4 L=60 d=32 9.9 and 11.3; per
// position B=500 80.0 and 73.6.  In the near form 31.7 and 32.9, 8.3 and 9.1; B=128 H=4 d=16 L=128 9.0 and 9.3, L=150 10.5 and 10.2, d=32 L=100
// 12.1 and 12.2, L=128 13.2 and 12.9; per position B=250 38.4 and 31.9).
// Short heads end before the order is found, and the more heads a CU takes one after another the more often it is found and the less
// it gives, so both of them bound the length from which it is used (a training step, fp32, lengths U[L/10,L], by length / in turn, us):
//   units          300                    600                    1200                   1800
//   d = 8   L=60   26.6 / 26.6   L=100   41.8 / 41.0   L=100   61.7 / 61.2   L=130   92.6 / 90.8
//          L=100   31.6 / 32.2   L=130   46.8 / 48.3   L=130   67.9 / 69.3   L=200  110.9 / 113.7
//   d = 16  L=60   27.8 / 27.9    L=60   37.8 / 37.6    L=60   54.3 / 53.3   L=100   91.8 / 89.6
//          L=100   34.3 / 35.7   L=100   45.6 / 46.0   L=100   67.4 / 68.6   L=130  109.4 / 110.2
//   d = 32  L=60   36.3 / 37.3    L=60   47.9 / 50.7    L=60   73.4 / 74.5    L=60  100.2 / 97.7
//          L=200   67.4 / 77.5   L=200   95.4 / 110.6  L=200  160 / 175      L=100  140.4 / 141.1
//   per position, in both passes
//           L=40   41.6 / 42.5    L=40   56.0 / 55.3    L=70  103.9 / 101.7  L=100  161 / 158
//           L=70   49.8 / 53.3    L=70   70.1 / 72.1   L=100  118.3 / 120.7  L=130  189 / 191
// The near form with eight wavefronts:
//           400 heads              600                   1000                  1600
//   d = 8   L=60   22.9 / 22.1   L=150   37.8 / 39.0   L=300   78.8 / 88.8
//          L=100   27.8 / 28.5
//   d = 16  L=60   24.2 / 23.9   L=150   43.0 / 45.7
//          L=100   30.2 / 31.6
//   d = 32  L=60   30.8 / 31.8   L=100   54.3 / 57.5   L=100   70.4 / 73.0   L=100   108 / 105
//          L=200   58.4 / 71.2   L=200   78.4 / 86.9   L=200    107 / 121    L=150   136 / 142
//   per position
//           L=60   32.5 / 32.2   L=150   61.3 / 68.7
//          L=100   40.5 / 48.6
// and with four:
//   d = 8                         L=60   24.6 / 24.3    L=60   27.6 / 27.6    L=60  38.2 / 37.2
//                                L=100   32.5 / 35.1   L=100   38.8 / 40.5   L=100  53.7 / 55.5
//   d = 16                        L=60   25.8 / 26.3    L=60   29.4 / 29.7    L=60  41.1 / 40.7
//                                L=100   35.5 / 39.0   L=100   43.6 / 45.8   L=100  60.0 / 62.0
//   d = 32                        L=60   33.9 / 35.3    L=60   40.0 / 41.6    L=60  57.3 / 60.3
//   per position                  L=60   35.1 / 37.8    L=60   42.9 / 44.2    L=60  60.0 / 61.6
int shortest_ordered(const KParams &p, int units, bool perpos, bool near)
{
  if (near && res_waves(p, units, true) == 4) return perpos ? 50 : p.d == 32 ? 45 : 50 + units / 40;
  if (near && p.d == 32 && !perpos) return 25 + units / 16;
  return perpos ? 30 + units / 18 : p.d == 32 ? 30 + units / 25 : (p.d == 16 ? 60 : 80) + units / 20;
}
bool order_by_length(const KParams &p, int units, bool perpos, bool near)
{
  return units > kCUs && !many_heads(units) && p.B <= kOrderRows && p.L >= shortest_ordered(p, units, perpos, near);
}
// per_simd: wavefronts a SIMD holds of a kernel whose tiles cost about the same (dQ of the near form).  Its workgroups then come in
// the number that ends together: rounds of the chip times a wavefront's tiles and its start, half a tile.  (us, by the first rule / so:
// B=16 H=8 L=1500 d=16 44.5 / 38.0, B=24 H=8 L=700 d=16 29.9 / 28.1, B=32 H=8 L=2000 d=8 63.2 / 63.9.  dK/dV, whose walks differ, 82.4 / 87.0
// there, and the forward at B=24 L=700 19.9 / 20.9: not for those.)
SmallPlan stream_plan(const KParams &p, int units, size_t words_per_wave, int per_simd = 0)
{
  const int NT = (p.L + kTile - 1) / kTile;
  SmallPlan s{false, false, kStreamWaves, 1, kStreamWaves * words_per_wave * sizeof(float)};
  if (per_simd > 0) {
    s.parts = parts_that_end_together(units, NT, s.waves, kCUs * per_simd);
    return s;
  }
  // enough workgroups for about two rounds of the chip's wavefronts (20 per CU), at most one tile per wavefront
  const int want = (2 * kCUs * 20 + units * s.waves - 1) / (units * s.waves);
  s.parts = std::max(1, std::min((NT + s.waves - 1) / s.waves, want));
  return s;
}
SmallPlan fwd_plan(const KParams &p, int dtype, bool perpos, int hpg, bool near)
{
  const size_t rows = (size_t)(p.L + kTile - 1) / kTile * kTile;
  const int units = p.B * p.H / hpg;
  SmallPlan s{true, false, res_waves(p, units, near), 1, 0};
  s.lds = (2 * rows * lds_row(dtype == 1, p.d) + (size_t)s.waves * lt_words(p, perpos)) * sizeof(float);
  if (p.nq == p.NB && s.lds <= small_lds_limit(p)) return s;
  s = stream_plan(p, p.B * p.H, lt_words(p, perpos));
  if (p.nq != p.NB) s = SmallPlan{false, false, 1, 1, lt_words(p, perpos) * sizeof(float)};  // serving mode: one query tile per head
  return s;
}
SmallPlan bwd_plan(const KParams &p, int dtype, bool perpos, int hpg)
{
  const int units = p.B * p.H / hpg;
  // with many heads four small workgroups per CU beat two that hold everything (B=2048 H=8 L=200 d=16: 672 against 917 us); with so
  // few that no CU has more than two to hold, everything fits beside a second one (gradients at B=82 H=4 L=174 d=16: 50.8 us with
  // everything in LDS, 52.3 with Q and dO read again; B=40 H=8 L=170 d=16, a whole step 47.5 and 48.4.  Whole steps in the near form: 749 against
  // 946, 34.6 and 35.4, 35.2 and 35.8; B=128 H=4 d=8 L=350 48.3 and 49.0)
  // A limit is about what both forms hold; the near form's gate rows and sums, 1 to 9 KB, come on top as long as the same number of
  // workgroups fits a CU.  (Counted in, they sent the longest heads the other way: a training step, us, in LDS / streamed, fp32 at L=240 with
  // B=64 H=8 d=16 52.6 / 62.7, B=125 H=8 d=16 87.1 / 95.5, per position with B=64 H=4 d=32 101 / 112, bf16 at B=600 H=4 L=416 d=32 404 / 466;
  // per position with 256 key/value heads at d=8 L=464 and d=16 L=400 120 / 117 and 105 / 102.)
  auto fits = [&](SmallPlan &s, size_t limit) {
    const ResLayout lay(p, lds_row(dtype == 1, p.d), perpos, hpg, s.overlay, s.waves);
    s.lds = (size_t)lay.total * sizeof(float);
    return (size_t)lay.held * sizeof(float) <= limit && s.lds <= (limit == kTwoPerCU ? 79 * 1024 : 52 * 1024);
  };
  for (int overlay = many_heads(units) ? 1 : 0; overlay < 2; ++overlay) {
    SmallPlan s{true, overlay != 0, res_waves(p, units, near_form(p)), 1, 0};
    if (!fits(s, small_lds_limit(p))) continue;
    SmallPlan all{true, false, s.waves, 1, 0};
    return s.overlay && units <= 2 * kCUs && fits(all, kTwoPerCU) ? all : s;
  }
  return stream_plan(p, p.B * p.H, lt_words(p, perpos), near_form(p) ? (p.d == 8 ? 5 : 4) : 0);
}

// The per-position form has limits that its callers know (144 KB of fp32 rows of 20 or 36 floats, see the header).
constexpr size_t kPosLimit = 144 * 1024;
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
void with_small_dims(const KParams &p, F &&f)
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

template <typename T>
static void launch_fwd_small_t(const KParams &p, const FwdArgs &a, hipStream_t st)
{
  const bool perpos = a.kv_groups > 0;
  const int hpg = perpos ? p.H / a.kv_groups : 1;
  const bool near = near_form(p) && !a.dense;
  const SmallPlan pl = fwd_plan(p, std::is_same<T, float>::value ? 0 : 1, perpos, hpg, near);
  const int grid = p.B * p.H / (pl.res ? hpg : 1) * pl.parts;
  with_small_dims(p, [&](auto dim, auto bk) {
    constexpr int D = decltype(dim)::value, BK = decltype(bk)::value;
    auto go = [&](auto kernel) {
      want_lds(kernel, pl.lds);
      hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(64 * pl.waves), pl.lds, st, (const T *)a.Q, (const T *)a.K,
                         (const T *)a.V, a.valid_len, a.dense ? nullptr : a.sel, a.gate_w, a.gate_b, (T *)a.O,
                         (float *)a.o_lt, (float *)a.o_st, a.lse_lt, a.lse_st, hpg, pl.parts, p);
    };
    const int shortest = !near ? 128 : p.d == 32 ? 112 : 150;
    const bool ordered = pl.res && order_by_length(p, grid, perpos, near) && (perpos || (grid <= 2 * kCUs && p.L >= shortest));
    if (near) {
      const NearMasks nm = near_masks(p, false);
      auto go = [&](auto kernel) {
        want_lds(kernel, pl.lds);
        hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(64 * pl.waves), pl.lds, st, (const T *)a.Q, (const T *)a.K,
                           (const T *)a.V, a.valid_len, a.sel, a.gate_w, a.gate_b, (T *)a.O, (float *)a.o_lt, (float *)a.o_st,
                           a.lse_lt, a.lse_st, hpg, pl.parts, nm, p);
      };
      if (ordered) perpos ? go(fwd_near_kernel<T, D, BK, true, true, true>) : go(fwd_near_kernel<T, D, BK, false, true, true>);
      else if (perpos) pl.res ? go(fwd_near_kernel<T, D, BK, true, true, false>) : go(fwd_near_kernel<T, D, BK, true, false, false>);
      else pl.res ? go(fwd_near_kernel<T, D, BK, false, true, false>) : go(fwd_near_kernel<T, D, BK, false, false, false>);
      return;
    }
    if (ordered)
      perpos ? go(fwd_small_kernel<T, D, BK, true, true, true>) : go(fwd_small_kernel<T, D, BK, false, true, true>);
    else if (perpos) pl.res ? go(fwd_small_kernel<T, D, BK, true, true, false>) : go(fwd_small_kernel<T, D, BK, true, false, false>);
    else pl.res ? go(fwd_small_kernel<T, D, BK, false, true, false>) : go(fwd_small_kernel<T, D, BK, false, false, false>);
  });
}

template <typename T>
static void launch_bwd_small_t(const KParams &p, const BwdArgs &a, const SmallWs &w, unsigned stages, int kv_groups, hipStream_t st)
{
  const bool perpos = kv_groups > 0;
  const int hpg = perpos ? p.H / kv_groups : 1;
  if ((stages & (kBwdStageGate | kBwdStageDQ | kBwdStageDKV)) == 0) return;
  const SmallPlan pl = bwd_plan(p, std::is_same<T, float>::value ? 0 : 1, perpos, hpg);
  with_small_dims(p, [&](auto dim, auto bk) {
    constexpr int D = decltype(dim)::value, BK = decltype(bk)::value;
    if (pl.res) {
      auto go = [&](auto kernel) {
        want_lds(kernel, pl.lds);
        hipLaunchKernelGGL(kernel, dim3((unsigned)(p.B * p.H / hpg)), dim3(64 * pl.waves), pl.lds, st, (const T *)a.Q,
                           (const T *)a.K, (const T *)a.V, a.valid_len, a.sel, a.gate_w, a.gate_b, (const float *)a.o_lt,
                           (const float *)a.o_st, a.lse_lt, a.lse_st, (const T *)a.dO, (T *)a.dQ, (T *)a.dK, (T *)a.dV, w.partial,
                           hpg, (int)pl.overlay, stages, p);
      };
      if (near_form(p)) {
        const NearMasks nm_q = near_masks(p, false), nm_k = near_masks(p, true);
        auto go = [&](auto kernel) {
          want_lds(kernel, pl.lds);
          hipLaunchKernelGGL(kernel, dim3((unsigned)(p.B * p.H / hpg)), dim3(64 * pl.waves), pl.lds, st, (const T *)a.Q,
                             (const T *)a.K, (const T *)a.V, a.valid_len, a.sel, a.gate_w, a.gate_b, (const float *)a.o_lt,
                             (const float *)a.o_st, a.lse_lt, a.lse_st, (const T *)a.dO, (T *)a.dQ, (T *)a.dK, (T *)a.dV, w.partial,
                             hpg, (int)pl.overlay, stages, nm_q, nm_k, p);
        };
        if (order_by_length(p, p.B * p.H / hpg, perpos, true)) perpos ? go(bwd_near_kernel<T, D, BK, true, true>) : go(bwd_near_kernel<T, D, BK, false, true>);
        else perpos ? go(bwd_near_kernel<T, D, BK, true, false>) : go(bwd_near_kernel<T, D, BK, false, false>);
        return;
      }
      if (order_by_length(p, p.B * p.H / hpg, perpos, false)) perpos ? go(bwd_res_kernel<T, D, BK, true, true>) : go(bwd_res_kernel<T, D, BK, false, true>);
      else perpos ? go(bwd_res_kernel<T, D, BK, true, false>) : go(bwd_res_kernel<T, D, BK, false, false>);
      return;
    }
    if (near_form(p)) {
      if (stages & (kBwdStageGate | kBwdStageDQ)) {
        auto go = [&](auto kernel) {
          hipLaunchKernelGGL(kernel, dim3((unsigned)(p.B * p.H * pl.parts)), dim3(64 * pl.waves), pl.lds, st, (const T *)a.Q,
                             (const T *)a.K, (const T *)a.V, a.valid_len, a.sel, a.gate_w, a.gate_b, (const float *)a.o_lt,
                             (const float *)a.o_st, a.lse_lt, a.lse_st, (const T *)a.dO, (T *)a.dQ, w, hpg, pl.parts, stages,
                             near_masks(p, false), p);
        };
        perpos ? go(bwd_dq_near_kernel<T, D, BK, true>) : go(bwd_dq_near_kernel<T, D, BK, false>);
        if (launch_failed()) return;
      }
      if (stages & kBwdStageDKV) {
        const SmallPlan pk = stream_plan(p, p.B * p.H / hpg, 0);
        auto go = [&](auto kernel) {
          hipLaunchKernelGGL(kernel, dim3((unsigned)(p.B * p.H / hpg * pk.parts)), dim3(64 * pk.waves), 0, st, (const T *)a.Q,
                             (const T *)a.K, (const T *)a.V, a.valid_len, a.gate_w, (const T *)a.dO, w, (T *)a.dK, (T *)a.dV, hpg,
                             pk.parts, near_masks(p, true), p);
        };
        perpos ? go(bwd_dkv_near_kernel<T, D, BK, true>) : go(bwd_dkv_near_kernel<T, D, BK, false>);
      }
      return;
    }
    if (stages & (kBwdStageGate | kBwdStageDQ)) {
      auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)(p.B * p.H * pl.parts)), dim3(64 * pl.waves), pl.lds, st, (const T *)a.Q,
                           (const T *)a.K, (const T *)a.V, a.valid_len, a.sel, a.gate_w, a.gate_b, (const float *)a.o_lt,
                           (const float *)a.o_st, a.lse_lt, a.lse_st, (const T *)a.dO, (T *)a.dQ, w, hpg, pl.parts, stages, p);
      };
      if (perpos) go(bwd_dq_small_kernel<T, D, BK, true>);
      else go(bwd_dq_small_kernel<T, D, BK, false>);
      if (launch_failed()) return;
    }
    if (stages & kBwdStageDKV) {
      const SmallPlan pk = stream_plan(p, p.B * p.H / hpg, 0);
      auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)(p.B * p.H / hpg * pk.parts)), dim3(64 * pk.waves), 0, st, (const T *)a.Q,
                           (const T *)a.K, (const T *)a.V, a.valid_len, a.gate_w, (const T *)a.dO, w, (T *)a.dK, (T *)a.dV, hpg,
                           pk.parts, p);
      };
      if (perpos) go(bwd_dkv_small_kernel<T, D, BK, true>);
      else go(bwd_dkv_small_kernel<T, D, BK, false>);
    }
  });
}

#ifdef BLOSSOM_SMALL_BF16
void launch_fwd_small_bf16(const KParams &p, const FwdArgs &a, hipStream_t st) { launch_fwd_small_t<bf16_t>(p, a, st); }
void launch_bwd_small_bf16(const KParams &p, const BwdArgs &a, const SmallWs &w, unsigned stages, int kv_groups, hipStream_t st)
{
  launch_bwd_small_t<bf16_t>(p, a, w, stages, kv_groups, st);
}
#else
bool small_supported(const KParams &p) { return small_shape(p); }

bool fwd_positions_supported(const KParams &p)
{
  return small_shape(p) && !p.bidir && p.NB <= 64 && p.nq == p.NB && pos_fwd_limit_bytes(p) <= kPosLimit;
}
bool bwd_positions_supported(const KParams &p) { return fwd_positions_supported(p) && pos_bwd_limit_bytes(p) <= kPosLimit; }

size_t small_ws_bytes(const KParams &p, SmallWs *w, char *base)
{
  if (!small_shape(p)) return 0;
  const size_t BH = (size_t)p.B * p.H, NT = (size_t)(p.L + kTile - 1) / kTile;
  const size_t NWt = (NT + 31) / 32, NWb = ((size_t)p.NB + 31) / 32;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char *at = base + off;
    off += (bytes + 255) & ~(size_t)255;
    return at;
  };
  w->rowc = reinterpret_cast<float *>(take(BH * NT * 6 * kTile * sizeof(float)));
  w->tile_words = reinterpret_cast<unsigned *>(take(BH * NT * NWt * sizeof(unsigned)));
  const size_t per_tile = std::max(p.b < kTile ? 2 * NWb : (size_t)1, bwd_positions_supported(p) ? (size_t)2 * kTile : (size_t)0);
  w->sel_bits = reinterpret_cast<unsigned *>(take(BH * NT * per_tile * sizeof(unsigned)));
  w->partial = reinterpret_cast<float *>(take(BH * NT * (2 * p.d + 1) * sizeof(float)));  // (at most one row per tile)
  return off;
}
int small_partial_rows(const KParams &p, int dtype, int kv_groups)
{
  return bwd_plan(p, dtype, kv_groups > 0, kv_groups > 0 ? p.H / kv_groups : 1).parts;
}

void launch_fwd_small(const KParams &p, int dtype, const FwdArgs &a, hipStream_t st)
{
  if (dtype == 0) launch_fwd_small_t<float>(p, a, st);
  else launch_fwd_small_bf16(p, a, st);
}

// gate pass and dQ, then dK/dV; kv_groups > 0: a.sel holds one row per position and group
void launch_bwd_small(const KParams &p, int dtype, const BwdArgs &a, const SmallWs &w, unsigned stages, int kv_groups,
                      hipStream_t st)
{
  if (dtype == 0) launch_bwd_small_t<float>(p, a, w, stages, kv_groups, st);
  else launch_bwd_small_bf16(p, a, w, stages, kv_groups, st);
}
#endif

}  // namespace blossom
