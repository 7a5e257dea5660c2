// Backward on the matrix cores for bf16, d = 64, block size 32 or 64: dQ (query-block
// stationary) and dK/dV (key-block stationary), chain rule through Eq. 1 and Eq. 16-19 with
// the selection held fixed.
//
// The upstream gradient of branch x is a_x*(dO + y_x*Wg_x) (a_lt = alpha, a_st = 1-alpha; gate backward, y_x per row): the caller's
// dO, a factor and a rank-one term.  It is never formed in memory.  With P' = a_x*P (log2(a_x) goes into the exponent)
//   dS_ij = P'_ij * (dO_i.v_j + y_i*u_j - D_i),  u_j = Wg_x.v_j,  D_i = (dO_i + y_i*Wg_x).o_x,i
//   dV_j = sum_i P'_ij dO_i + (sum_i P'_ij y_i) Wg_x,   dK_j = sum_i dS_ij q_i,   dQ_i = sum_j dS_ij k_j
// In dK/dV dO enters as it is, and the rank-one term to 2^-17: the cancellation that rows with one or two keys rely on
// (dO.v_j + y*u_j = D when P = 1) survives.  In dQ, where a lane keeps its row, the bracket dO + y_x*Wg_x is rounded to bf16 once and
// its row constant c_x is taken with the same rounded values.  With two rounded gradients in memory and residual passes of dK/dV for
// rows with few keys a training step at B=128 H=4 L=1024 k=8 w=64 in blocks of 32 took 345 us (the per-row pass 62, these kernels
// 190) instead of 309 (47, 178), at B=32 H=8 L=1997 with all of Eq. 15 488 instead of 467.  At B=16 H=8 L=8192 k=16 w=128 in
// blocks of 64, 2012 instead of 1999 (181 and 1206 against 130 and 1230), it is even but for what two boxes differ by: sixteen more
// additions a unit for the sums of P'*y.  dK and dV came out with 5 % larger errors.
//
// Accumulators start at minus a per-row constant, so the MFMA result is directly what the next
// step needs: the exponent S'' = c*q.k - lse*log2(e) + log2(a_x) (Q or K pre-multiplied by c =
// scale*log2(e)) and the bracket of dS.  The constants arrive as three-term bf16 splits (exact), y as two terms.
// dK/dV, where they change with every query tile, brings them into the accumulator by one
// extra matrix instruction (row terms x ones, and x the terms of u_j); dQ, where a lane keeps its row for the whole walk,
// holds them as two 16-register blocks that the first matrix instruction of each product
// takes as its C operand.  Either way no per-element VALU initialisation is needed.  (Reading
// the dK/dV constants from LDS straight into a C block was measured slower: that kernel
// already issues 25 LDS reads per 18 matrix instructions.)  Probabilities and dS leave the accumulator
// registers as the B operand of the next product without moving between lanes; the matching
// A operands (K^T, Q^T, dO^T) come from LDS through the transposing ds_read_b64_tr_b16.
// Query blocks whose rows may see only a few keys (large probabilities) feed P and dS as
// two-term bf16 sums.
//
// Matrix pipe and vector ALUs share the issue and are busy 85 % of the time together, so what a tile does not need is left out:
// masks are bits (two instructions an element instead of four; three of the six one-launch kernels shed their four spilled registers,
// the one with mask blocks smaller than its tile of 32 keeps its sixteen), and at block 64 a unit of 32 keys (queries) none of
// the wavefront's rows sees (keys are seen by) is skipped.  A training step at B=16 H=8 L=8192 k=16 w=128 2078 -> 2042 us with both, at
// B=128 H=4 L=1024 k=8 w=64 in blocks of 32 403 -> 398 us.
#include "gate_reduce.h"
#include "launch.h"
#include "mfma_common.h"

// x * y, and zero where either is zero, whatever the other: the padding's values may be any finite ones, whose products overflow, and no
// infinity is to meet a probability of zero.  (v_mul_legacy_f32, as the compiler's intrinsic: in assembly it would not wait for a
// matrix instruction's result.  Dropping the products of padded keys by a mask instead: a training step at B=64 H=8 L=500 b=64, lengths
// U[50,500], 195.3 us; with this 192.4, as without either.)
__device__ float mul_or_zero(float x, float y) __asm("llvm.amdgcn.fmul.legacy");

namespace blossom {

using namespace mfma;

namespace {

// Per-lane LDS BYTE offsets of the two operand read patterns for a tile staged with swz().
// Kept in bytes and passed through an empty asm by the kernels, so that "tile base + offset +
// constant" is formed next to each read and the constant folds into the instruction's immediate.
struct ReadOffsets {
  int row[4];  // row-per-lane 16-byte reads: slab kk; add 2*32*unit*D
  int tr[2];   // transposing 8-byte reads: M-block mb; add 2*(32*unit + 16*t)*D
  int tr8[2];  // the same for the read 8 rows further down (row bit 3 set: another swizzle)
};

__device__ __forceinline__ ReadOffsets read_offsets(int lane)
{
  ReadOffsets o;
  const int lq = lane & 31, lh = lane >> 5, r16 = lane & 15, g1 = (lane >> 4) & 1;
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) o.row[kk] = 2 * (lq * D + (((2 * kk + lh) ^ swz(lq)) * 8));
#pragma unroll
  for (int mb = 0; mb < 2; ++mb)
  {
    const int row = 4 * lh + (r16 >> 2);  // rows row and row + 8 of a 16-row contraction slab
    const int chunk = 4 * mb + 2 * g1 + ((r16 & 3) >> 1);
    o.tr[mb] = 2 * (row * D + ((chunk ^ swz(row)) * 8) + 4 * (r16 & 1));
    o.tr8[mb] = 2 * ((row + 8) * D + ((chunk ^ swz(row + 8)) * 8) + 4 * (r16 & 1));
  }
  return o;
}

// Direct global->LDS staging of one tile (BLK rows x 128 bytes): each wavefront moves 4 x 1 KB.
// A tile's rows are contiguous in memory and the LDS copy keeps the 128-byte row pitch, so one
// uniform base (SGPRs), one per-lane byte offset and the same immediate on the global and the
// LDS side address the four 8-row slices.
template <int BLK>
struct Stager {
  int wv, ld_row;
  bool ragged;
  int L, NB;
  unsigned lane_off;  // bytes: (ld_row, chunk) of this lane inside a tile (BLK = 32: the chunk alone), 8-row slices 0 and 2
  unsigned lane_odd;  // the same for slices 1 and 3 (row bit 3 set: another swizzle)
  __device__ __forceinline__ void init(int wv_, int lane, int L_, int NB_)
  {
    wv = wv_;
    L = L_;
    NB = NB_;
    ld_row = 32 * wv + (lane >> 3);
    ragged = L % BLK != 0;
    // LDS chunk position lane&7 holds chunk (lane&7)^swz(row)
    lane_off = (unsigned)((BLK == 32 ? 0 : ld_row * D) + ((lane & 7) ^ swz(ld_row)) * 8) * 2u;
    lane_odd = (unsigned)((BLK == 32 ? 0 : ld_row * D) + ((lane & 7) ^ swz(ld_row + 8)) * 8) * 2u;
  }
  // src_head: first element of the (row, head) slice of the tensor
  __device__ __forceinline__ void stage(const uint16_t *src_head, uint16_t *dst_tile, int blk) const
  {
    constexpr int TILE = BLK * D;
    if constexpr (BLK == 32) {
      // (no branch for the last, partial block: its rows past the end are clamped, always masked; a buffer load, for the
      // compiler counts the global one as a flat access, before which it waits for everything: see REFILL)
      const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(src_head), 0, L * (D * 2), 0x00020000);
      const int row_max = L - 1 - blk * BLK;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const unsigned off = (unsigned)min(ld_row + 8 * u, row_max) * (D * 2) + ((u & 1) ? lane_odd : lane_off);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(src, (lds_void *)(dst_tile + 8 * u * D), 16, off, blk * (TILE * 2), 0, 0);
      }
      return;
    }
    const char *src = reinterpret_cast<const char *>(src_head) + (size_t)max(blk, 0) * (TILE * 2);  // uniform (block -1: a skipped list entry, not read)
    lds_void *dst = (lds_void *)(dst_tile + 32 * wv * D);
    if (!ragged || blk != NB - 1) {
      __builtin_amdgcn_global_load_lds((glb_void *)(src + lane_off), dst, 16, 0, 0);
      __builtin_amdgcn_global_load_lds((glb_void *)(src + lane_odd), dst, 16, 1024, 0);
      __builtin_amdgcn_global_load_lds((glb_void *)(src + lane_off), dst, 16, 2048, 0);
      __builtin_amdgcn_global_load_lds((glb_void *)(src + lane_odd), dst, 16, 3072, 0);
    } else {  // last, partial block: rows past the end are clamped (always masked)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int over = max(0, blk * BLK + ld_row + 8 * u - (L - 1));
        const unsigned off = ((u & 1) ? lane_odd : lane_off) + (unsigned)((8 * u - over) * D * 2);
        __builtin_amdgcn_global_load_lds((glb_void *)(src + off), (lds_void *)(dst_tile + (32 * wv + 8 * u) * D), 16, 0, 0);
      }
    }
  }
};

// off: byte offset inside the tile
__device__ __forceinline__ bf16x8 lds_row(const uint16_t *tile, int off)
{
  return *reinterpret_cast<const bf16x8 *>(reinterpret_cast<const char *>(tile) + off);
}

__device__ __forceinline__ bf16x8 lds_tr(const uint16_t *tile, int off, int off8)
{
  const char *a = reinterpret_cast<const char *>(tile);
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(a + off));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(a + off8));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// 16 accumulator values -> two bf16 B operands (contraction halves t = 0, 1)
__device__ __forceinline__ void to_operand(const f32x16 &a, bf16x8 (&f)[2])
{
#pragma unroll
  for (int i = 0; i < 16; i += 2) {
    const bf16x2 pk = {(__bf16)a[i], (__bf16)a[i + 1]};
    f[i >> 3][i & 7] = pk[0];
    f[i >> 3][(i & 7) + 1] = pk[1];
  }
}

// row of bf16 (this lane's 4 slabs of 8) as the stationary operand
__device__ __forceinline__ void load_frags(const uint16_t *row, int lh, bf16x8 (&f)[4])
{
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) f[kk] = *reinterpret_cast<const bf16x8 *>(row + 16 * kk + 8 * lh);
}
// ... times c (apart from the loads, so that other requests go out before their arrival is waited for)
__device__ __forceinline__ void scale_frags(float c, bf16x8 (&f)[4])
{
#pragma unroll
  for (int kk = 0; kk < 4; ++kk)
#pragma unroll
    for (int e = 0; e < 8; ++e) f[kk][e] = (__bf16)((float)f[kk][e] * c);
}

// Stores 2 x 16 accumulators (d x rows, transposed) as bf16, scaled, through LDS: the wavefront's 32 rows
// (this lane: row lane%32, channels
// 32*mb + 8*g + 4*(lane/32) + e in acc[mb][4*g + e]) are written into its own 4 KB of staging rows
// (free once the walk is over; chunks XOR-swizzled against bank conflicts) and leave as whole
// 128-byte rows, 8 rows per store instruction, non-temporal (nothing in this library reads the
// gradients back).  Rows that are not kept are stored as zeros, rows at or past rows_left not at all.
// `unrope` (dQ and dK when the caller's Q and K went through the rotary position embedding): the rows
// are rotated back first; a lane's four consecutive channels are two whole channel pairs.  m_row0 is
// the position of the first of the 32 rows, L the sequence length (rows past it are never stored).
__device__ __forceinline__ void store_rows_bf16(uint16_t *dst_row0, int rows_left, uint16_t *pt, const f32x16 (&acc)[2],
                                                float scale, bool keep, const KParams &p, bool unrope = false, int m_row0 = 0)
{
  int el;  // the lane id, rebuilt here so that none of the addressing below is computed ahead of the walk
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(el));
  const int elq = el & 31, elh = el >> 5;
  const float sc = keep ? scale : 0.0f;
  const bool rot = unrope && p.rope_cos != nullptr;
  auto put = [&](int mb, int g, float v0, float v1, float v2, float v3) __attribute__((always_inline)) {
    uint2 pk;
    pk.x = pack2_bf16(v0 * sc, v1 * sc);
    pk.y = pack2_bf16(v2 * sc, v3 * sc);
    const int chunk = 4 * mb + g;  // 16-byte chunk of the row; this lane fills half elh of it
    *reinterpret_cast<uint2 *>(pt + elq * D + ((chunk ^ (elq & 7)) * 8) + 4 * elh) = pk;
  };
  if (rot) {  // (its own branch around all of it, the tables requested eight pairs at a time)
    const size_t first = (size_t)min(m_row0 + elq, p.L - 1) * (D / 2) + 2 * elh;
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
      float2 c[4], s[4];  // channels 32*mb + 8*g + 4*elh + (0..3) are the pairs 16*mb + 4*g + 2*elh + (0, 1)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        c[g] = *reinterpret_cast<const float2 *>(p.rope_cos + first + 16 * mb + 4 * g);
        s[g] = *reinterpret_cast<const float2 *>(p.rope_sin + first + 16 * mb + 4 * g);
      }
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float v0 = acc[mb][4 * g], v1 = acc[mb][4 * g + 1], v2 = acc[mb][4 * g + 2], v3 = acc[mb][4 * g + 3];
        unrope_pair(c[g].x, s[g].x, v0, v1);
        unrope_pair(c[g].y, s[g].y, v2, v3);
        put(mb, g, v0, v1, v2, v3);
      }
    }
  } else {
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g) put(mb, g, acc[mb][4 * g], acc[mb][4 * g + 1], acc[mb][4 * g + 2], acc[mb][4 * g + 3]);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int rr = 8 * i + (el >> 3), c = el & 7;
    const uint4 v = *reinterpret_cast<const uint4 *>(pt + rr * D + ((c ^ (rr & 7)) * 8));
    typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
    const u32x4_t vv = {v.x, v.y, v.z, v.w};
    if (rr < rows_left) __builtin_nontemporal_store(vv, reinterpret_cast<u32x4_t *>(dst_row0 + (size_t)rr * D + 8 * c));
  }
}

// s_waitcnt immediates (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8)
constexpr int vmcnt_imm(int n) { return (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); }  // all but the n youngest
constexpr int kVm0 = vmcnt_imm(0);                     // every vector-memory operation has finished
constexpr int kLgkm0 = 15 | (7 << 4) | (3 << 14);      // every LDS and scalar-memory operation has

constexpr int kFewKeys = 32;    // rows seeing fewer keys than this get two-term bf16 operands

// A row's constants (bwd_prep_kernel) are an MFMA operand as they are loaded, s0 s1 | D2 s2 | D0 D1 | y0 y1, in both halves of the
// wavefront.  What they meet picks the exponent's constant, or -D and y times the lane's u_j = Wg_x.v_j (two terms, one in each half: as
// exact as y).  Slots that are not meant meet zeros and have to be finite.
__device__ __forceinline__ bf16x8 row_operand(const uint4 &r) { return __builtin_bit_cast(bf16x8, r); }
__device__ __forceinline__ bf16x8 exponent_columns(int lh)
{
  constexpr uint32_t one = 0x3F80u;
  return __builtin_bit_cast(bf16x8, lh == 0 ? make_uint4(one | one << 16, one << 16, 0u, 0u) : make_uint4(0u, 0u, 0u, 0u));
}
__device__ __forceinline__ bf16x8 bracket_columns(float u, int lh)
{
  constexpr uint32_t one = 0x3F80u;
  const uint32_t t = split2(u), term = lh == 0 ? t & 0xFFFFu : t >> 16;
  return __builtin_bit_cast(bf16x8, make_uint4(0u, lh == 0 ? one : 0u, lh == 0 ? one | one << 16 : 0u, term | term << 16));
}

// Where the sixteen rows of a lane's accumulator are found in its row of 16 lanes: lane l holds the value of tile row acc_row(l), and
// sum_rows adds sum_i P[i] * value(row of P[i]) with the value as a DPP operand (row_newbcast), without a register for each.
__device__ __forceinline__ int acc_row(int lane) { return 8 * ((lane >> 2) & 3) + 4 * (lane >> 5) + (lane & 3); }
// (In assembly: the compiler makes sixteen moves of it.  A DPP operand may be read two states after it was written.)
__device__ __forceinline__ void sum_rows(const f32x16 &P, float x, float &sum)
{
#define ROW(n) "\n\tv_fmac_f32_dpp %0, %1, %" #n " row_newbcast:"
#define ALL " row_mask:0xf bank_mask:0xf"
  asm("s_nop 1" ROW(2) "0" ALL ROW(3) "1" ALL ROW(4) "2" ALL ROW(5) "3" ALL ROW(6) "4" ALL ROW(7) "5" ALL ROW(8) "6" ALL ROW(9) "7" ALL
      ROW(10) "8" ALL ROW(11) "9" ALL ROW(12) "10" ALL ROW(13) "11" ALL ROW(14) "12" ALL ROW(15) "13" ALL ROW(16) "14" ALL ROW(17) "15" ALL
      : "+v"(sum)
      : "v"(x), "v"(P[0]), "v"(P[1]), "v"(P[2]), "v"(P[3]), "v"(P[4]), "v"(P[5]), "v"(P[6]), "v"(P[7]), "v"(P[8]), "v"(P[9]), "v"(P[10]),
        "v"(P[11]), "v"(P[12]), "v"(P[13]), "v"(P[14]), "v"(P[15]));
#undef ALL
#undef ROW
}

// this lane's 32 channels of a branch's gate weights (the slabs of load_frags)
__device__ __forceinline__ void load_gate(const float *w, int lh, float (&g)[4][8])
{
#pragma unroll
  for (int kk = 0; kk < 4; ++kk)
#pragma unroll
    for (int e = 0; e < 8; e += 4) load4(w + 16 * kk + 8 * lh + e, reinterpret_cast<float(&)[4]>(g[kk][e]));
}

}  // namespace

// =============================================================================================
// dQ: one workgroup per (row, head, query block), one wavefront per 32 query rows.
//   per 32-key unit:  S''^T = K (cQ)^T - lse2       (keys x queries, lane owns a query column)
//                     G^T   = V (dO + y_x*Wg_x)^T - c_x
//                     dS^T  = 2^S'' * G^T  -> bf16 -> B operand
//                     dQ^T += K^T dS^T      (K^T through the transposing LDS read)
// EQ15: the short-term mask is all of Eq. 15, with mask block BLK or (SUB) a power of two below it;
// compile-time variants of both kernels, so that the plain window keeps its code.
// =============================================================================================
// (pid: the workgroup's index among the dQ workgroups of the launch; Ks0..Vs1: four staging tiles of BLK*D halfwords
// in LDS, 1 KB aligned, distinct objects)
template <int BLK, bool EQ15, bool SUB>
__device__ __forceinline__ void bwd_dq_body(
    const uint16_t *__restrict__ Q, const uint16_t *__restrict__ K, const uint16_t *__restrict__ V,
    const int *__restrict__ valid_len, const int *__restrict__ sel, const uint4 *__restrict__ rowI_lt,
    const uint4 *__restrict__ rowI_st, const uint16_t *__restrict__ dO, const float4 *__restrict__ rowstat, const float *__restrict__ gate_w,
    const float *__restrict__ o_lt, const float *__restrict__ o_st, uint16_t *__restrict__ dQ, KParams p, unsigned pid,
    uint16_t *Ks0, uint16_t *Ks1, uint16_t *Vs0, uint16_t *Vs1)
{
  constexpr int UNITS = BLK / 32;
  constexpr bool ONE = UNITS == 1;  // a workgroup of one wavefront: see REFILL at bwd_both_mfma_kernel

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: MFMA regions must be scalar branches
  const int lq = lane & 31, lh = lane >> 5;
  const unsigned vid = xcd_spread(pid, (unsigned)(p.B * p.H), (unsigned)p.NB);
  const int bh = (int)(vid / p.NB);
  const int I = p.NB - 1 - (int)(vid % p.NB);
  const int n = clamp_len(valid_len[bh / p.H], p.L);
  const int p0 = p.L - n;
  const int q0 = I * BLK + 32 * wv;
  const int iq = q0 + lq;
  const bool q_ok = iq < p.L && iq >= p0;
  const size_t head = (size_t)bh * p.L * D;
  const size_t rowoff = head + (size_t)min(iq, p.L - 1) * D;
  const size_t lrow = (size_t)bh * p.L + min(iq, p.L - 1);

  f32x16 dq[2];
#pragma unroll
  for (int i = 0; i < 16; ++i) { dq[0][i] = 0.0f; dq[1][i] = 0.0f; }
  if (min((I + 1) * BLK, p.L) <= p0) {  // no valid query: gradients are zero
    zero_rows(dQ + head, q0, 32, p.L, lane);
    return;
  }

  bf16x8 qf[4], gf[4], gf_next[4];  // gf: the short-term bracket (the walk starts with the window tiles), gf_next: the long-term one
  load_frags(Q + rowoff, lh, qf);
  load_frags(dO + rowoff, lh, gf);
  const float *gate = gate_w + (size_t)(bh % p.H) * 2 * D;
  float w_lt[4][8], w_st[4][8];
  load_gate(gate, lh, w_lt);
  load_gate(gate + D, lh, w_st);
  const float4 rs = rowstat[lrow];  // y_lt, y_st, -c_lt, -c_st; zeros in a pad row of a block with a valid one
  // per-row constants (pad rows carry an exponent of -1e30: every probability of the column is zero)
  const uint4 ri_st = rowI_st[lrow];
  const uint4 ri_lt = rowI_lt[lrow];
  // s_init, g_init: -lse2[i] (with log2(a_x)) and -c_x[i] of this lane's row in every accumulator slot.  The
  // first matrix instruction of each product takes them as its C operand, so the logits and
  // dP - c_x leave the matrix cores with the row terms already applied.
  f32x16 s_init, g_init;
  auto set_init = [&](uint32_t sx, uint32_t sy, float b) __attribute__((always_inline)) {
    const float a = unsplit3(sx, sy >> 16);
#pragma unroll
    for (int i = 0; i < 16; ++i) { s_init[i] = a; g_init[i] = b; }
    asm volatile("" : "+v"(s_init), "+v"(g_init));  // register blocks, not one value copied at each use
  };

  // ---- tile list: window blocks, then the selection list up to its last valid entry ----
  const int J_first = p0 / BLK;
  const int lowpos = I * BLK - (p.w - 1);
  int J_lo = lowpos <= 0 ? 0 : lowpos / BLK;
  // SUB: the mask block of Eq. 15 is a power of two below BLK.  The mask-block distances 2^r below
  // one tile then reach into block I - 1, which joins the window range; the larger ones land on
  // the blocks I - 2^r' as before; every short-term tile is masked element by element.
  constexpr bool sub = EQ15 && SUB;
  const int sub_sh = sub ? __builtin_ctz((unsigned)p.sblk) : 0;
  if (sub) J_lo = min(J_lo, I - 1);
  J_lo = max(J_lo, J_first);
  // With the full short-term mask (Eq. 15) the blocks I - 2^r below the window
  // range follow the window blocks: r = r0 .. r0 + n_pow - 1.
  const int n_win = I - J_lo + 1;
  int n_st = n_win, r0 = 0;
  if (EQ15 && I > J_first) {
    const int d_win = I - J_lo;                                      // largest block distance inside the window range
    r0 = d_win == 0 ? 0 : 32 - __builtin_clz((unsigned)d_win);       // smallest r with 2^r > d_win
    const int r_max = 31 - __builtin_clz((unsigned)(I - J_first));   // largest r with I - 2^r >= J_first
    n_st += max(0, r_max - r0 + 1);
  }
  int n_lt = 0;
  bool lt_few = true;  // the selected past blocks hold fewer than kFewKeys valid keys
  const int *my_sel = sel + ((size_t)bh * p.NB + I) * p.k;
  // (entries outside [0, NB) are skipped wherever they stand: the walk runs up to the last valid
  // entry, an invalid one in between costs one tile with every key masked)
  for (int e0 = 0; e0 < p.k; e0 += 64) {
    const int e = e0 + lane;
    const int J = e < p.k ? my_sel[e] : -1;
    const bool ok = J >= 0 && J < p.NB;
    const unsigned long long okm = __ballot(ok);
    if (okm != 0ull) n_lt = e0 + 64 - __builtin_clzll(okm);
    const int vcount = min((J + 1) * BLK, p.L) - max(J * BLK, p0);
    if (__ballot(ok && J < I && vcount >= kFewKeys) != 0ull) lt_few = false;
  }
  // Rows with only a few keys: dq is a sum of a few large dS*k terms that nearly cancel, so the
  // bf16 rounding of dS would dominate it.  Such wavefronts feed dS as a two-term bf16 sum.
  const int hp_st = __builtin_amdgcn_readfirstlane((int)(p.w < kFewKeys || q0 - p0 + 1 < kFewKeys));
  const int hp_lt = __builtin_amdgcn_readfirstlane((int)lt_few);
  const int n_all = n_st + n_lt;
  // For those rows the bf16 rounding of the bracket itself would show as well (dS is large, and the
  // small projections of it on v_j - o lose relative accuracy): its residual enters as a second B operand, and the row constant
  // gains the matching residual.o_x.
  bf16x8 gl[4], gl_next[4];
  float c1_lt = rs.z, c1_st = rs.w;
#pragma unroll
  for (int kk = 0; kk < 4; ++kk)
#pragma unroll
    for (int e = 0; e < 8; ++e) { gl[kk][e] = (__bf16)0.0f; gl_next[kk][e] = (__bf16)0.0f; }
  if (hp_st | hp_lt) {
    bf16x8 dof[4];
    load_frags(dO + rowoff, lh, dof);
    auto residual = [&](const float *w, float y, const float *o_row, bf16x8 (&lo)[4]) __attribute__((always_inline)) -> float {
      float corr = 0.0f;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        float g[8], o[8];
#pragma unroll
        for (int e = 0; e < 8; e += 4) {
          load4(w + 16 * kk + 8 * lh + e, reinterpret_cast<float(&)[4]>(g[e]));
          load4(o_row + 16 * kk + 8 * lh + e, reinterpret_cast<float(&)[4]>(o[e]));
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float full = fmaf(y, g[e], (float)dof[kk][e]);
          lo[kk][e] = (__bf16)(q_ok ? full - (float)(__bf16)full : 0.0f);
          corr = fmaf((float)lo[kk][e], o[e], corr);
        }
      }
      return q_ok ? corr + __shfl_xor(corr, 32) : 0.0f;
    };
    c1_lt -= residual(gate, rs.x, o_lt + rowoff, gl_next);
    c1_st -= residual(gate + D, rs.y, o_st + rowoff, gl);
  }
  if constexpr (!ONE) __syncthreads();
  // Block id of tile t: window blocks by arithmetic, selected blocks by a scalar load from the
  // selection row (uniform address), issued a whole tile before its value is needed.
  auto tile_of = [&](int t) -> int {
    const int e = __builtin_amdgcn_readfirstlane(t - n_st);
    typedef const int __attribute__((address_space(4))) *const_int_ptr;  // read-only: loads become scalar
    if (e >= 0) return ((const_int_ptr)my_sel)[e];  // raw: may be outside [0, NB), see list_entry
    if (!EQ15) return J_lo + t;
    return t < n_win ? J_lo + t : I - (1 << (r0 + t - n_win));
  };

  // a raw tile-list value when it is consumed (a whole tile after its scalar load was issued): entries
  // outside [0, NB), blocks after the query block and blocks of nothing but padding, whose values may be anything, become -1, a
  // tile whose keys are all masked and which holds the rows of the own block
  auto list_entry = [&](int raw) -> int { return (unsigned)(raw - J_first) <= (unsigned)(I - J_first) ? raw : -1; };

  Stager<BLK> sg;
  sg.init(wv, lane, p.L, p.NB);
  const uint16_t *k_lane = K + head;  // (row, head) slices; the stager adds block and lane offsets
  const uint16_t *v_lane = V + head;
  ReadOffsets ro = read_offsets(lane);
  auto stage_tile = [&](uint16_t *ks, uint16_t *vs, int J) __attribute__((always_inline)) {
    if (ONE) J = J < 0 ? I : J;
    sg.stage(k_lane, ks, J);
    sg.stage(v_lane, vs, J);
  };

  // (refill: called once the tile has been read to registers, ONE only)
  auto tile_body = [&](const uint16_t *ks, const uint16_t *vs, int J, bool short_term, auto refill) __attribute__((always_inline)) {
    asm volatile("" : "+v"(ro.row[0]), "+v"(ro.row[1]), "+v"(ro.row[2]), "+v"(ro.row[3]), "+v"(ro.tr[0]), "+v"(ro.tr[1]), "+v"(ro.tr8[0]), "+v"(ro.tr8[1]));
    const bool hp = (short_term ? hp_st : hp_lt) != 0;
    // band-masked by the window, unless Eq. 15 shows the whole block (power-of-two block distance)
    const bool windowed = short_term && !(EQ15 && !sub && is_pow2(I - J));
    const bool masked = windowed || J == I || J * BLK < p0;
    int wlo = iq - p.w + 1;
    if (EQ15 && iq >= p.last_lo) wlo = min(wlo, p.last_lo);  // third case of Eq. 15: the last block is visible to its own rows
    const int lo = windowed ? max(p0, wlo) : p0;
    const unsigned span = (unsigned)(iq - lo);
    const bool any = iq >= lo;
#pragma unroll
    for (int s = 0; s < UNITS; ++s) {
      if constexpr (!ONE) {  // no row of the wavefront sees any of the 32 keys: later than all of them, padding, a skipped entry, below the window
        const int k_lo = J * BLK + 32 * s, k_hi = k_lo + 31;
        if (J < 0 || k_lo > q0 + 31 || k_hi < p0 || (!EQ15 && windowed && k_hi < q0 - p.w + 1)) continue;
      }
      bf16x8 kt[2][2];  // K^T operands of the last product
      auto read_kt = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int mb = 0; mb < 2; ++mb) kt[t][mb] = lds_tr(ks, 2 * (32 * s + 16 * t) * D + ro.tr[mb], 2 * (32 * s + 16 * t) * D + ro.tr8[mb]);
      };
      f32x16 sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_row(ks, 2 * 32 * s * D + ro.row[0]), qf[0], s_init, 0, 0, 0);
      f32x16 gacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_row(vs, 2 * 32 * s * D + ro.row[0]), gf[0], g_init, 0, 0, 0);
#pragma unroll
      for (int kk = 1; kk < 4; ++kk) {
        sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_row(ks, 2 * 32 * s * D + ro.row[kk]), qf[kk], sacc, 0, 0, 0);
        gacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_row(vs, 2 * 32 * s * D + ro.row[kk]), gf[kk], gacc, 0, 0, 0);
      }
      if (hp) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
          gacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_row(vs, 2 * 32 * s * D + ro.row[kk]), gl[kk], gacc, 0, 0, 0);
      }
      if constexpr (ONE) {
        read_kt();
        __builtin_amdgcn_s_waitcnt(kLgkm0);
        refill();
      }
      if (masked) {
        const int base = J * BLK + 32 * s + 4 * lh;
        if (sub && windowed && J < J_lo && J * BLK >= p0) {
          // a block I - 2^r' below the window range, all of it valid: visible iff row and key share
          // the mask block within their tiles (no window, no last-block key, one possible power of two)
          const int qo = iq & (BLK - 1);
          const int kb = 32 * s + 4 * lh;
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int ko = kb + 8 * (i >> 2) + (i & 3);
            sacc[i] = (((qo ^ ko) >> sub_sh) == 0 && q_ok) ? sacc[i] : kNegInf;
          }
        } else if (sub && windowed) {
          // window range, or (valid, causal and) a power-of-two mask-block distance, or a last-block key
          const unsigned cspan = (unsigned)(iq - p0);
          const bool cany = iq >= p0;
          const int qmb = iq >> sub_sh;
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int key = base + 8 * (i >> 2) + (i & 3);
            const int x = qmb - (key >> sub_sh);
            const bool far = cany & ((unsigned)(key - p0) <= cspan) & ((x > 0 && (x & (x - 1)) == 0) | (key >= p.last_lo));
            const bool vis = (any & ((unsigned)(key - lo) <= span)) | far;
            sacc[i] = vis ? sacc[i] : kNegInf;
          }
        } else {
          keep_rows(sacc, row_bits(lo - J * BLK - 32 * s, iq - J * BLK - 32 * s), lh, kNegInf);
        }
      }
#pragma unroll
      for (int i = 0; i < 16; ++i)  // dS
        sacc[i] = mul_or_zero(__builtin_amdgcn_exp2f(sacc[i]), gacc[i]);
      bf16x8 dsf[2];
      to_operand(sacc, dsf);
      if constexpr (!ONE) read_kt();
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) dq[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kt[t][mb], dsf[t], dq[mb], 0, 0, 0);
      if (hp) {
#pragma unroll
        for (int i = 0; i < 16; ++i) sacc[i] -= (float)dsf[i >> 3][i & 7];
        to_operand(sacc, dsf);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int mb = 0; mb < 2; ++mb) dq[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kt[t][mb], dsf[t], dq[mb], 0, 0, 0);
      }
    }
  };

  auto to_long_term = [&]() __attribute__((always_inline)) {  // the long-term tiles start: that branch's gradient and constants
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      gf[kk] = gf_next[kk];
      gl[kk] = gl_next[kk];
    }
    set_init(ri_lt.x, ri_lt.y, c1_lt);
  };
  int J_cur = list_entry(tile_of(0));
  int J_nxt = list_entry(tile_of(min(1, n_all - 1)));
  stage_tile(Ks0, Vs0, J_cur);
  if constexpr (ONE) {
    __builtin_amdgcn_sched_barrier(0);  // (the first tile's loads stay the older ones: what the loop's waits count on)
    stage_tile(Ks1, Vs1, J_nxt);
    __builtin_amdgcn_sched_barrier(0);
  }
  scale_frags(p.scale * kLog2e, qf);
  // the brackets; zeros in a pad row, where dO may hold anything and y is zero
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    uint4 raw = __builtin_bit_cast(uint4, gf[kk]);
    raw = make_uint4(q_ok ? raw.x : 0u, q_ok ? raw.y : 0u, q_ok ? raw.z : 0u, q_ok ? raw.w : 0u);
    const bf16x8 g8 = __builtin_bit_cast(bf16x8, raw);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      gf_next[kk][e] = (__bf16)fmaf(rs.x, w_lt[kk][e], (float)g8[e]);
      gf[kk][e] = (__bf16)fmaf(rs.y, w_st[kk][e], (float)g8[e]);
    }
  }
  set_init(ri_st.x, ri_st.y, c1_st);
  if constexpr (ONE) {
    int J_2 = list_entry(tile_of(min(2, n_all - 1)));
    auto step = [&](int t, uint16_t *ks, uint16_t *vs) __attribute__((always_inline)) {
      const int J_after = tile_of(min(t + 3, n_all - 1));  // consumed at the end of this step
      if (t == n_st) to_long_term();
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(8));  // the tile is there; the next one's eight loads may be on their way
      tile_body(ks, vs, J_cur, t < n_st, [&]() __attribute__((always_inline)) { stage_tile(ks, vs, J_2); });
      J_cur = J_nxt;
      J_nxt = J_2;
      J_2 = list_entry(J_after);
    };
    int t = 0;
    for (; t + 1 < n_all; t += 2) {
      step(t, Ks0, Vs0);
      step(t + 1, Ks1, Vs1);
    }
    if (t < n_all) step(t, Ks0, Vs0);
    __builtin_amdgcn_s_waitcnt(kVm0);  // (the last two refills are not read, but they write LDS)
  } else {
    __syncthreads();
    auto step = [&](int t, uint16_t *k_fill, uint16_t *v_fill, const uint16_t *k_cur, const uint16_t *v_cur)
                    __attribute__((always_inline)) {
      const int J_after = tile_of(min(t + 2, n_all - 1));  // consumed at the end of this step
      if (t + 1 < n_all) stage_tile(k_fill, v_fill, J_nxt);
      if (t == n_st) to_long_term();
      tile_body(k_cur, v_cur, J_cur, t < n_st, [] {});
      J_cur = J_nxt;
      J_nxt = list_entry(J_after);
      __syncthreads();
    };
    for (int t = 0; t < n_all; t += 2) {
      step(t, Ks1, Vs1, Ks0, Vs0);
      if (t + 1 < n_all) step(t + 1, Ks0, Vs0, Ks1, Vs1);
    }
  }
  {  // (every wavefront is past the last barrier of the walk: the staging rows are free)
    const int row0 = I * BLK + 32 * wv;
    store_rows_bf16(dQ + head + (size_t)row0 * D, p.L - row0, Ks0 + wv * 32 * D, dq, p.scale, q_ok, p, true, row0);
  }
}

// =============================================================================================
// dK, dV: one workgroup per (row, head, key block), one wavefront per 32 key rows; walks the
// query blocks whose window reaches the key block, then those that selected it (inverse list).
//   per 32-query unit:  S'' = Q (cK)^T - lse2[i] + log2(a_x[i])   (queries x keys, lane owns a key column)
//                       G   = dO V^T + y_x[i]*u_x[j] - D_x[i]
//                       P' = 2^S'',  dS = P'*G
//                       dV^T += dO^T P',  dK^T += Q^T dS,  r_x[j] += sum_i P'*y_x[i]
//   and at the end dV^T += Wg_lt r_lt + Wg_st r_st
// =============================================================================================

template <int BLK, bool EQ15, bool SUB>
__device__ __forceinline__ void bwd_dkv_body(
    const uint16_t *__restrict__ Q, const uint16_t *__restrict__ K, const uint16_t *__restrict__ V,
    const int *__restrict__ valid_len, const uint4 *__restrict__ rowI_lt, const uint4 *__restrict__ rowI_st,
    const int *__restrict__ offs, const int *__restrict__ items, const uint16_t *__restrict__ dO,
    const float *__restrict__ gate_w, uint16_t *__restrict__ dK, uint16_t *__restrict__ dV, KParams p, unsigned pid,
    uint16_t *Qs0, uint16_t *Qs1, uint16_t *Gs0, uint16_t *Gs1, uint4 *rc0, uint4 *rc1)
{
  // (rc0, rc1: 64 row constants each, of the staged query tiles)
  constexpr int UNITS = BLK / 32;
  constexpr bool ONE = UNITS == 1;  // a workgroup of one wavefront: see REFILL at bwd_both_mfma_kernel

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 31, lh = lane >> 5;
  const unsigned vid = xcd_spread(pid, (unsigned)(p.B * p.H), (unsigned)p.NB);
  const int bh = (int)(vid / p.NB);
  const int J = (int)(vid % p.NB);  // early key blocks are selected by more query blocks: start them first
  const int n = clamp_len(valid_len[bh / p.H], p.L);
  const int p0 = p.L - n;
  const int j = J * BLK + 32 * wv + lq;  // this lane's key row
  const bool key_ok = j < p.L && j >= p0;
  const size_t head = (size_t)bh * p.L * D;
  const size_t rowoff = head + (size_t)min(j, p.L - 1) * D;
  const size_t lbase = (size_t)bh * p.L;

  f32x16 dk[2], dv[2];
#pragma unroll
  for (int i = 0; i < 16; ++i) { dk[0][i] = 0.0f; dk[1][i] = 0.0f; dv[0][i] = 0.0f; dv[1][i] = 0.0f; }
  if (min((J + 1) * BLK, p.L) <= p0) {  // no valid key
    zero_rows(dK + head, J * BLK + 32 * wv, 32, p.L, lane);
    zero_rows(dV + head, J * BLK + 32 * wv, 32, p.L, lane);
    return;
  }
  bf16x8 kf[4], vf[4];
  load_frags(K + rowoff, lh, kf);
  load_frags(V + rowoff, lh, vf);
  const float *gate = gate_w + (size_t)(bh % p.H) * 2 * D;

  // ---- walk: window part I = J..I_hi, then the inverse selection list ----
  const long last_q = (long)J * BLK + (BLK - 1) + (p.w - 1);
  // SUB: the mask block of Eq. 15 is a power of two below BLK: block J + 1 joins the window range (the
  // mask-block distances below one tile reach it), every short-term tile is masked element by element.
  constexpr bool sub = EQ15 && SUB;
  const int sub_sh = sub ? __builtin_ctz((unsigned)p.sblk) : 0;
  int I_hi = (int)min((long)(p.NB - 1), last_q / BLK);
  if (sub) I_hi = max(I_hi, min(J + 1, p.NB - 1));
  // With the full short-term mask (Eq. 15) the query blocks J + 2^r above the
  // window range follow: r = r0 .. r0 + n_pow - 1.
  const int n_win = I_hi - J + 1;
  int n_st = n_win, r0 = 0;
  if (EQ15 && p.NB - 1 > J) {
    const int d_win = I_hi - J;                                       // largest block distance inside the window range
    r0 = d_win == 0 ? 0 : 32 - __builtin_clz((unsigned)d_win);        // smallest r with 2^r > d_win
    const int r_max = 31 - __builtin_clz((unsigned)(p.NB - 1 - J));   // largest r with J + 2^r <= NB - 1
    n_st += max(0, r_max - r0 + 1);
  }
  const int e_lo = offs[(size_t)bh * (p.NB + 1) + J];
  const int n_lt = offs[(size_t)bh * (p.NB + 1) + J + 1] - e_lo;
  const int n_all = n_st + n_lt;
  const int *my_items = items + (size_t)bh * p.NB * p.k + e_lo;
  // Query block of step t, with the few-keys flag of the list entries in bit kInvFewShift:
  // window blocks by arithmetic, list entries by a scalar load (uniform address), issued a
  // whole tile before the value is needed.
  auto entry_of = [&](int t) -> int {
    const int e = __builtin_amdgcn_readfirstlane(t - n_st);
    typedef const int __attribute__((address_space(4))) *const_int_ptr;  // read-only: loads become scalar
    if (e >= 0) return ((const_int_ptr)my_items)[e];
    if (!EQ15) return J + t;
    return t < n_win ? J + t : J + (1 << (r0 + t - n_win));
  };

  Stager<BLK> sg;
  sg.init(wv, lane, p.L, p.NB);
  const uint16_t *q_lane = Q + head;  // (row, head) slices; the stager adds block and lane offsets
  const uint16_t *g_lane = dO + head;
  ReadOffsets ro = read_offsets(lane);
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const uint4 pad_consts = make_uint4(0x0000f149u, 0u, 0u, 0u);  // -1e30 as (hi, 0, 0): probability zero

  // per-row constants of query block Iq for one branch (rows past the end: probability zero)
  auto row_consts = [&](int Iq, bool windowed) __attribute__((always_inline)) -> uint4 {
    uint4 r = pad_consts;
    if (tid < BLK) {
      const int i = Iq * BLK + tid;
      if (i < p.L) r = (windowed ? rowI_st : rowI_lt)[lbase + i];
    }
    return r;
  };

  const bf16x8 s_terms = exponent_columns(lh);
  bf16x8 u_terms;                  // of the branch the walk is in, short-term first
  float u_lt;
  float r_sum = 0.0f, r_st = 0.0f;  // this lane's part of r_x, of the branch the walk is in and of the short-term one
  auto gate_products = [&]() __attribute__((always_inline)) {
    if (J * BLK < p0) {  // the products of a padded key's value may overflow
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const uint4 v = __builtin_bit_cast(uint4, vf[kk]);
        vf[kk] = __builtin_bit_cast(bf16x8, make_uint4(key_ok ? v.x : 0u, key_ok ? v.y : 0u, key_ok ? v.z : 0u, key_ok ? v.w : 0u));
      }
    }
    auto product = [&](const float *w) __attribute__((always_inline)) -> float {
      float g[4][8], u = 0.0f;
      load_gate(w, lh, g);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
#pragma unroll
        for (int e = 0; e < 8; ++e) u = fmaf(g[kk][e], (float)vf[kk][e], u);
      return u + __shfl_xor(u, 32);
    };
    u_lt = product(gate);
    u_terms = bracket_columns(product(gate + D), lh);
  };
  auto to_long_term = [&]() __attribute__((always_inline)) {
    u_terms = bracket_columns(u_lt, lh);
    r_st = r_sum;
    r_sum = 0.0f;
  };

  // (rcs: the tile's row constants; refill: called once the tile has been read to registers, ONE only)
  auto tile_body = [&](const uint16_t *qs, uint16_t *gsm, const uint4 *rcs, int Iq, bool short_term, bool hp,
                       auto refill) __attribute__((always_inline)) {
    // band-masked by the window, unless Eq. 15 shows the whole block (power-of-two block distance)
    const bool windowed = short_term && !(EQ15 && !sub && is_pow2(Iq - J));
    asm volatile("" : "+v"(ro.row[0]), "+v"(ro.row[1]), "+v"(ro.row[2]), "+v"(ro.row[3]), "+v"(ro.tr[0]), "+v"(ro.tr[1]), "+v"(ro.tr8[0]), "+v"(ro.tr8[1]));
    const bool masked = windowed || Iq == J || Iq * BLK < p0 || J * BLK < p0 || (Iq + 1) * BLK > p.L;
    // visible <=> key valid and lo_i <= i <= hi_i
    const int lo_i = max(j, p0);
    // (third case of Eq. 15: a key among the last block's positions is visible to every later row)
    const int hi_i = windowed && !(EQ15 && j >= p.last_lo) ? min(p.L - 1, j + p.w - 1) : p.L - 1;
    const unsigned span = (unsigned)(hi_i - lo_i);
    const bool any = key_ok && hi_i >= lo_i;
    if (Iq * BLK < p0) {  // dO is the caller's in the padding too, where a product may overflow (either wavefront writes the same zeros)
      if constexpr (ONE) __builtin_amdgcn_s_waitcnt(kVm0);
      for (int o = 16 * lane; o < (p0 - Iq * BLK) * (D * 2); o += 1024)
        *reinterpret_cast<uint4 *>(reinterpret_cast<char *>(gsm) + o) = make_uint4(0u, 0u, 0u, 0u);
    }
#pragma unroll
    for (int s = 0; s < UNITS; ++s) {
      if constexpr (!ONE) {  // none of the 32 query rows sees a key of the wavefront: earlier than all of them, padding, past the window
        const int i_lo = Iq * BLK + 32 * s, i_hi = i_lo + 31, j0 = J * BLK + 32 * wv;
        if (i_hi < j0 || i_hi < p0 || j0 + 31 < p0 || (!EQ15 && windowed && i_lo > j0 + 31 + p.w - 1)) continue;
      }
      const uint4 rc = rcs[32 * s + lq];
      const uint32_t y = rcs[32 * s + acc_row(lane)].w;
      bf16x8 gt[2][2], qt[2][2];  // dO^T and Q^T operands of the last products
      auto read_tr = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int mb = 0; mb < 2; ++mb) {
            gt[t][mb] = lds_tr(gsm, 2 * (32 * s + 16 * t) * D + ro.tr[mb], 2 * (32 * s + 16 * t) * D + ro.tr8[mb]);
            qt[t][mb] = lds_tr(qs, 2 * (32 * s + 16 * t) * D + ro.tr[mb], 2 * (32 * s + 16 * t) * D + ro.tr8[mb]);
          }
      };
      f32x16 sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(row_operand(rc), s_terms, zero16, 0, 0, 0);
      f32x16 gacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(row_operand(rc), u_terms, zero16, 0, 0, 0);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_row(qs, 2 * 32 * s * D + ro.row[kk]), kf[kk], sacc, 0, 0, 0);
        gacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_row(gsm, 2 * 32 * s * D + ro.row[kk]), vf[kk], gacc, 0, 0, 0);
      }
      if constexpr (ONE) {
        read_tr();
        __builtin_amdgcn_s_waitcnt(kLgkm0);
        refill();
      }
      if (masked) {
        const int base = Iq * BLK + 32 * s + 4 * lh;
        if (sub && windowed && Iq > I_hi && (Iq + 1) * BLK <= p.L) {
          // a whole query block J + 2^r' above the window range: visible iff row and key share the mask
          // block within their tiles (no window; a last-block key lies in the last two blocks, whose
          // rows are all inside the window range of their own and the previous block)
          const int jo = j & (BLK - 1);
          const int qb = 32 * s + 4 * lh;
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int qio = qb + 8 * (i >> 2) + (i & 3);
            sacc[i] = (((jo ^ qio) >> sub_sh) == 0 && key_ok) ? sacc[i] : kNegInf;
          }
        } else if (sub && windowed) {
          // window range, or (valid, causal and) a power-of-two mask-block distance, or a last-block key
          const unsigned cspan = (unsigned)(p.L - 1 - lo_i);
          const int kmb = j >> sub_sh;
          const bool last = j >= p.last_lo;
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int qi = base + 8 * (i >> 2) + (i & 3);
            const int x = (qi >> sub_sh) - kmb;
            const bool far = key_ok & ((unsigned)(qi - lo_i) <= cspan) & ((x > 0 && (x & (x - 1)) == 0) | last);
            const bool vis = (any & ((unsigned)(qi - lo_i) <= span)) | far;
            sacc[i] = vis ? sacc[i] : kNegInf;
          }
        } else {
          keep_rows(sacc, row_bits(lo_i - Iq * BLK - 32 * s, key_ok ? hi_i - Iq * BLK - 32 * s : -1), lh, kNegInf);
        }
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        sacc[i] = __builtin_amdgcn_exp2f(sacc[i]);  // P'
        gacc[i] *= sacc[i];                         // dS
      }
      bf16x8 pf[2], dsf[2];
      to_operand(sacc, pf);
      to_operand(gacc, dsf);
      if constexpr (!ONE) read_tr();
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) {
          dv[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(gt[t][mb], pf[t], dv[mb], 0, 0, 0);
          dk[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qt[t][mb], dsf[t], dk[mb], 0, 0, 0);
        }
      sum_rows(sacc, unsplit2(y), r_sum);
      if (hp) {  // rows with few keys: large P and dS, add the rounding residuals as a second bf16 term
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          sacc[i] -= (float)pf[i >> 3][i & 7];
          gacc[i] -= (float)dsf[i >> 3][i & 7];
        }
        to_operand(sacc, pf);
        to_operand(gacc, dsf);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int mb = 0; mb < 2; ++mb) {
            dv[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(gt[t][mb], pf[t], dv[mb], 0, 0, 0);
            dk[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qt[t][mb], dsf[t], dk[mb], 0, 0, 0);
          }
      }
    }
  };

  // rows that may see fewer than kFewKeys keys: the first valid rows of a window (or a very
  // short window), or a query block flagged by the inverse list
  auto few = [&](int ent, bool win) -> bool {
    return win ? (p.w < kFewKeys || (ent & kInvBlockMask) * BLK - p0 + 1 < kFewKeys) : (ent >> kInvFewShift) != 0;
  };
  int ent_cur = entry_of(0);
  int ent_nxt = entry_of(min(1, n_all - 1));
  if constexpr (ONE) {
    // (the row constants go straight to LDS too, ten registers less; rows past the end take the last one's, and are masked)
    auto fill = [&](uint16_t *qs, uint16_t *gsm, uint4 *rc, int ent, bool win) __attribute__((always_inline)) {
      const int Iq = ent & kInvBlockMask;
      sg.stage(q_lane, qs, Iq);
      sg.stage(g_lane, gsm, Iq);
      const uint4 *src_head = (win ? rowI_st : rowI_lt) + lbase;
      const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4 *>(src_head), 0, p.L * (int)sizeof(uint4), 0x00020000);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(src, (lds_void *)rc, 16, (unsigned)min(Iq * BLK + lq, p.L - 1) * (unsigned)sizeof(uint4), 0, 0, 0);
    };
    fill(Qs0, Gs0, rc0, ent_cur, 0 < n_st);
    __builtin_amdgcn_sched_barrier(0);  // (the first tile's loads stay the older ones: what the loop's waits count on)
    fill(Qs1, Gs1, rc1, ent_nxt, 1 < n_st);
    __builtin_amdgcn_sched_barrier(0);
    gate_products();
    scale_frags(p.scale * kLog2e, kf);
    int ent_2 = entry_of(min(2, n_all - 1));
    auto step = [&](int t, uint16_t *qs, uint16_t *gsm, uint4 *rc) __attribute__((always_inline)) {
      const int ent_after = entry_of(min(t + 3, n_all - 1));  // consumed at the end of this step
      const bool win = t < n_st;
      const int Iq = ent_cur & kInvBlockMask;
      if (t == n_st) to_long_term();
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(9));  // the tile is there; the next one's nine loads may be on their way
      tile_body(qs, gsm, rc, Iq, win, few(ent_cur, win), [&]() __attribute__((always_inline)) { fill(qs, gsm, rc, ent_2, t + 2 < n_st); });
      ent_cur = ent_nxt;
      ent_nxt = ent_2;
      ent_2 = ent_after;
    };
    int t = 0;
    for (; t + 1 < n_all; t += 2) {
      step(t, Qs0, Gs0, rc0);
      step(t + 1, Qs1, Gs1, rc1);
    }
    if (t < n_all) step(t, Qs0, Gs0, rc0);
    __builtin_amdgcn_s_waitcnt(kVm0);  // (the last two refills are not read, but they write LDS)
  } else {
    {
      const int I0 = ent_cur & kInvBlockMask;
      const bool win0 = 0 < n_st;
      sg.stage(q_lane, Qs0, I0);
      sg.stage(g_lane, Gs0, I0);
      const uint4 r0 = row_consts(I0, win0);
      gate_products();
      scale_frags(p.scale * kLog2e, kf);
      if (tid < BLK) rc0[tid] = r0;
    }
    __syncthreads();
    auto step = [&](int t, uint16_t *q_fill, uint16_t *g_fill, const uint16_t *q_cur, uint16_t *g_cur,
                    const uint4 *rc_cur, uint4 *rc_fill) __attribute__((always_inline)) {
      uint4 rn = pad_consts;
      const bool more = t + 1 < n_all;
      const int ent_after = entry_of(min(t + 2, n_all - 1));  // consumed at the end of this step
      if (more) {
        const int In = ent_nxt & kInvBlockMask;
        const bool win_n = t + 1 < n_st;
        rn = row_consts(In, win_n);
        sg.stage(q_lane, q_fill, In);
        sg.stage(g_lane, g_fill, In);
      }
      const bool win = t < n_st;
      if (t == n_st) to_long_term();
      tile_body(q_cur, g_cur, rc_cur, ent_cur & kInvBlockMask, win, few(ent_cur, win), [] {});
      if (more && tid < BLK) rc_fill[tid] = rn;
      ent_cur = ent_nxt;
      ent_nxt = ent_after;
      __syncthreads();
    };
    for (int t = 0; t < n_all; t += 2) {
      step(t, Qs1, Gs1, Qs0, Gs0, rc0, rc1);
      if (t + 1 < n_all) step(t + 1, Qs0, Gs0, Qs1, Gs1, rc1, rc0);
    }
  }

  // ---- the rank-one terms of dV ----
  if (n_all <= n_st) to_long_term();
  const float r_lt = r_sum + __shfl_xor(r_sum, 32);
  r_st += __shfl_xor(r_st, 32);
  // (As products of three-term splits, long-term in the lower half of the contraction, short-term in the upper one.  Two vector
  // instructions for each element, the weights loaded in that layout, a select for each element of dQ's brackets and a test for
  // each row constant were 6 % of the vector instructions at B=128 H=4 L=1024 k=8 w=64, and 333 instead of 327 us a training step.)
  {
    const uint2 r = split3(lh == 0 ? r_lt : r_st);
    const uint32_t rh = r.x & 0xFFFFu, rm = r.x >> 16, rl = r.y;
    const bf16x8 cols = __builtin_bit_cast(bf16x8, make_uint4(rh | rm << 16, rh | rm << 16, rl | rh << 16, 0u));
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
      const uint2 w = split3(gate[lh * D + 32 * mb + lq]);
      const uint32_t wh = w.x & 0xFFFFu, wm = w.x >> 16, wl = w.y;
      const bf16x8 rows = __builtin_bit_cast(bf16x8, make_uint4(wh | wh << 16, wm | wm << 16, wh | wl << 16, 0u));
      dv[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rows, cols, dv[mb], 0, 0, 0);
    }
  }

  {  // (every wavefront is past the last barrier of the walk: the staging rows are free)
    const int row0 = J * BLK + 32 * wv;
    store_rows_bf16(dK + head + (size_t)row0 * D, p.L - row0, Qs0 + wv * 32 * D, dk, p.scale, key_ok, p, true, row0);
    store_rows_bf16(dV + head + (size_t)row0 * D, p.L - row0, Gs0 + wv * 32 * D, dv, 1.0f, key_ok, p);
  }
}

#define BWD_LDS_TILES(BLK)                                                   \
  __shared__ __attribute__((aligned(1024))) uint16_t lds_t0[(BLK) * D];      \
  __shared__ __attribute__((aligned(1024))) uint16_t lds_t1[(BLK) * D];      \
  __shared__ __attribute__((aligned(1024))) uint16_t lds_t2[(BLK) * D];      \
  __shared__ __attribute__((aligned(1024))) uint16_t lds_t3[(BLK) * D]

#define BWD_DQ_PARAMS                                                                                              \
  const uint16_t *__restrict__ Q, const uint16_t *__restrict__ K, const uint16_t *__restrict__ V,                  \
      const int *__restrict__ valid_len, const int *__restrict__ sel, const uint4 *__restrict__ rowI_lt,           \
      const uint4 *__restrict__ rowI_st, const uint16_t *__restrict__ dO, const float4 *__restrict__ rowstat,      \
      const float *__restrict__ gate_w,                                                                            \
      const float *__restrict__ o_lt, const float *__restrict__ o_st, uint16_t *__restrict__ dQ
#define BWD_DQ_ARGS Q, K, V, valid_len, sel, rowI_lt, rowI_st, dO, rowstat, gate_w, o_lt, o_st, dQ
#define BWD_DKV_ARGS Q, K, V, valid_len, rowI_lt, rowI_st, offs, items, dO, gate_w, dK, dV

template <int BLK, bool EQ15, bool SUB>
__global__ __launch_bounds__(BLK * 2) __attribute__((amdgpu_waves_per_eu(2, 2))) void bwd_dq_mfma_kernel(BWD_DQ_PARAMS, KParams p)
{
  BWD_LDS_TILES(BLK);
  bwd_dq_body<BLK, EQ15, SUB>(BWD_DQ_ARGS, p, blockIdx.x, lds_t0, lds_t1, lds_t2, lds_t3);
}

template <int BLK, bool EQ15, bool SUB>
__global__ __launch_bounds__(BLK * 2) __attribute__((amdgpu_waves_per_eu(2, 2))) void bwd_dkv_mfma_kernel(
    const uint16_t *__restrict__ Q, const uint16_t *__restrict__ K, const uint16_t *__restrict__ V,
    const int *__restrict__ valid_len, const uint4 *__restrict__ rowI_lt, const uint4 *__restrict__ rowI_st,
    const int *__restrict__ offs, const int *__restrict__ items, const uint16_t *__restrict__ dO,
    const float *__restrict__ gate_w, uint16_t *__restrict__ dK, uint16_t *__restrict__ dV, KParams p)
{
  BWD_LDS_TILES(BLK);
  __shared__ __attribute__((aligned(1024))) uint4 lds_rc0[64];
  __shared__ __attribute__((aligned(1024))) uint4 lds_rc1[64];
  bwd_dkv_body<BLK, EQ15, SUB>(BWD_DKV_ARGS, p, blockIdx.x, lds_t0, lds_t1, lds_t2, lds_t3, lds_rc0, lds_rc1);
}

// workgroups that sum the partial gate gradients: kGateCols columns of a head each
constexpr int kGateCols = 8;
__host__ __device__ inline int gate_groups(const KParams &p) { return (2 * p.d + kGateCols) / kGateCols; }
inline unsigned gate_workgroups(const KParams &p) { return ((unsigned)(p.H * gate_groups(p)) + 7u) / 8u * 8u; }

// dQ and dK/dV in ONE launch (the full backward call): the first B*H*NB workgroups take the key blocks, the
// rest the query blocks.  The two kernels need the same workgroup shape, the same two wavefronts per SIMD and
// nearly the same LDS, so nothing is lost by the union, and the short dQ workgroups fill the slots that the
// tail of the skewed dK/dV walks leaves idle (and one launch gap goes).  Before them come `gate_wgs` workgroups, a multiple of 8 so
// that the others keep their XCDs, that sum the partial gate gradients (7.5 us as a launch of its own at B=128 H=4 L=1024; at
// block size 64 the walks come out slower beside that code, 1280 against 1240 us at B=16 H=8 L=8192, and it stays a launch of its own).
//
// REFILL.  At block size 32 a workgroup is one wavefront, its body of 12 or 18 matrix instructions is shorter than a
// load's latency under load, and LDS holds two tiles for each of the eight wavefronts of a CU.  So a tile is read to
// registers whole (the transposed operands too), and its buffer is refilled with the tile after next at once: a load
// has nearly two bodies to arrive.  The loop issues the same loads on every path and has one exit (an odd last tile is
// a step of its own), so that a wait at the head of a step counts exactly past the younger loads: a wait of the kernel's own, for
// the compiler does not reliably put one between loads to LDS and the reads of it.
// B=128 H=4 L=1024 k=8 w=64, lengths U[100,1024]: 230 -> 202 us; B=32 H=8 L=1997, all of Eq. 15: 267 -> 239 us.
template <int BLK, bool EQ15, bool SUB>
__global__ __launch_bounds__(BLK * 2) __attribute__((amdgpu_waves_per_eu(2, 2))) void bwd_both_mfma_kernel(
    BWD_DQ_PARAMS, const int *__restrict__ offs, const int *__restrict__ items, uint16_t *__restrict__ dK,
    uint16_t *__restrict__ dV, const float *__restrict__ partial, float *__restrict__ d_gate_w, float *__restrict__ d_gate_b, int nchunk,
    unsigned gate_wgs, KParams p)
{
  BWD_LDS_TILES(BLK);  // the four staging tiles serve either role
  __shared__ __attribute__((aligned(1024))) uint4 lds_rc0[64];
  __shared__ __attribute__((aligned(1024))) uint4 lds_rc1[64];
  if (BLK == 32 && blockIdx.x < gate_wgs) {
    const int groups = gate_groups(p), h = blockIdx.x / groups;
    if (h < p.H)
      gate_reduce<BLK * 2, kGateCols>(partial, d_gate_w, d_gate_b, nchunk, p, h, (blockIdx.x - h * groups) * kGateCols,
                                      reinterpret_cast<float(*)[kGateCols + 1]>(lds_t0));
    return;
  }
  const unsigned n = (unsigned)(p.B * p.H * p.NB), id = blockIdx.x - gate_wgs;
  if (id < n) bwd_dkv_body<BLK, EQ15, SUB>(BWD_DKV_ARGS, p, id, lds_t0, lds_t1, lds_t2, lds_t3, lds_rc0, lds_rc1);
  else bwd_dq_body<BLK, EQ15, SUB>(BWD_DQ_ARGS, p, id - n, lds_t0, lds_t1, lds_t2, lds_t3);
}

bool bwd_mfma_takes_gate(const KParams &p, unsigned stages)
{
  constexpr unsigned all = kBwdStageGate | kBwdStageDQ | kBwdStageDKV;
  return p.b == 32 && (stages & all) == all && 2ull * p.B * p.H * p.NB + gate_workgroups(p) <= 0x7FFFFFFFull;
}

bool bwd_mfma_supported(const KParams &p, int dtype)
{
  return dtype == 1 && p.d == 64 && (p.b == 32 || p.b == 64) && !p.bidir &&
         (p.sblk == 0 || (is_pow2(p.sblk) && p.sblk <= p.b));
}

void launch_bwd_mfma(const KParams &p, const BwdArgs &a, const BwdWorkspace &w, unsigned stages, hipStream_t st)
{
  const bool do_dq = stages & kBwdStageDQ, do_dkv = stages & kBwdStageDKV;
  const unsigned grid = (unsigned)(p.B * p.H * p.NB);
  auto u16 = [](const void *x) { return reinterpret_cast<const uint16_t *>(x); };
  auto go_dq = [&](auto kernel, unsigned threads) {
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, st, u16(a.Q), u16(a.K), u16(a.V), a.valid_len, a.sel,
                       w.rowI_lt, w.rowI_st, u16(a.dO), w.rowstat, a.gate_w, (const float *)a.o_lt,
                       (const float *)a.o_st, (uint16_t *)a.dQ, p);
  };
  auto go_dkv = [&](auto kernel, unsigned threads) {
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, st, u16(a.Q), u16(a.K), u16(a.V), a.valid_len, w.rowI_lt,
                       w.rowI_st, w.offs, w.items, u16(a.dO), a.gate_w, (uint16_t *)a.dK, (uint16_t *)a.dV, p);
  };
  const bool eq15 = p.sblk != 0;
  const bool sub = eq15 && p.sblk < p.b;  // mask block smaller than the tile
  if (do_dq && do_dkv && 2ull * grid <= 0x7FFFFFFFull) {
    const unsigned gate_wgs = bwd_mfma_takes_gate(p, stages) ? gate_workgroups(p) : 0u;
    auto go = [&](auto kernel, unsigned threads) {
      hipLaunchKernelGGL(kernel, dim3(2 * grid + gate_wgs), dim3(threads), 0, st, u16(a.Q), u16(a.K), u16(a.V), a.valid_len, a.sel,
                         w.rowI_lt, w.rowI_st, u16(a.dO), w.rowstat, a.gate_w, (const float *)a.o_lt,
                         (const float *)a.o_st, (uint16_t *)a.dQ, w.offs, w.items, (uint16_t *)a.dK, (uint16_t *)a.dV, w.partial, a.d_gate_w, a.d_gate_b,
                         w.nchunk, gate_wgs, p);
    };
    if (p.b == 32) {
      if (sub) go(bwd_both_mfma_kernel<32, true, true>, 64);
      else if (eq15) go(bwd_both_mfma_kernel<32, true, false>, 64);
      else go(bwd_both_mfma_kernel<32, false, false>, 64);
    } else {
      if (sub) go(bwd_both_mfma_kernel<64, true, true>, 128);
      else if (eq15) go(bwd_both_mfma_kernel<64, true, false>, 128);
      else go(bwd_both_mfma_kernel<64, false, false>, 128);
    }
    return;
  }
  if (p.b == 32) {
    if (do_dq) {
      if (sub) go_dq(bwd_dq_mfma_kernel<32, true, true>, 64);
      else if (eq15) go_dq(bwd_dq_mfma_kernel<32, true, false>, 64);
      else go_dq(bwd_dq_mfma_kernel<32, false, false>, 64);
      if (launch_failed()) return;
    }
    if (do_dkv) {
      if (sub) go_dkv(bwd_dkv_mfma_kernel<32, true, true>, 64);
      else if (eq15) go_dkv(bwd_dkv_mfma_kernel<32, true, false>, 64);
      else go_dkv(bwd_dkv_mfma_kernel<32, false, false>, 64);
    }
  } else {
    if (do_dq) {
      if (sub) go_dq(bwd_dq_mfma_kernel<64, true, true>, 128);
      else if (eq15) go_dq(bwd_dq_mfma_kernel<64, true, false>, 128);
      else go_dq(bwd_dq_mfma_kernel<64, false, false>, 128);
      if (launch_failed()) return;
    }
    if (do_dkv) {
      if (sub) go_dkv(bwd_dkv_mfma_kernel<64, true, true>, 128);
      else if (eq15) go_dkv(bwd_dkv_mfma_kernel<64, true, false>, 128);
      else go_dkv(bwd_dkv_mfma_kernel<64, false, false>, 128);
    }
  }
}

}  // namespace blossom
