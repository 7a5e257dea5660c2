// Types and small helpers shared by the matrix-core kernels (bf16, d = 64, gfx950).
#pragma once

#include "common.h"

namespace blossom {
namespace mfma {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef __attribute__((address_space(3))) void lds_void;
typedef const __attribute__((address_space(1))) void glb_void;

constexpr int D = 64;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kNegInf = -__builtin_huge_valf();

// Maps the hardware workgroup id (dealt round-robin over the 8 XCDs) to a virtual id in units of `per` ids each, a unit being what
// shares data (a head): all ids of a unit go to one XCD and meet in its L2, and units go to the XCDs in turn.  (Handing each XCD
// a contiguous range of units would give it whole batch rows, whose lengths differ: at B=32 H=8, lengths U[200,1997], the
// fullest XCD had a third more than the average to do and the others waited for it.)  The units beyond a multiple of 8 are
// spread over the XCDs in contiguous ranges of ids.
__device__ __forceinline__ unsigned xcd_spread(unsigned pid, unsigned units, unsigned per)
{
  constexpr unsigned X = 8;
  const unsigned whole = units / X * X * per, xcd = pid % X;
  if (pid < whole) {
    const unsigned local = pid / X, u = local / per;
    return (u * X + xcd) * per + (local - u * per);
  }
  const unsigned total = units % X * per, local = (pid - whole) / X;
  const unsigned tall_per = (total + X - 1) / X;  // ids of a "tall" XCD
  const unsigned tall = total % X ? total % X : X;
  return whole + (xcd < tall ? xcd * tall_per + local : tall * tall_per + (xcd - tall) * (tall_per - 1) + local);
}

// A staged tile is BLK rows of 128 bytes; 16-byte chunk c of row r sits at chunk position
// c ^ swz(r).  Measured on gfx950: the LDS serves 16 lanes x 16 bytes per cycle over 64 banks
// (rows of 128 bytes alternate between the two bank halves), and the lanes of one cycle of a
// 16-byte read run over bits 1-3 of the lane index (bit 4 tied to them, bit 0 free).  The
// swizzle serves both operand read patterns without bank conflicts:
//  - row-per-lane 16-byte reads (lane = row, one chunk column): swz is injective over row bits
//    1-3 for fixed bits 0 and 4 (position bits: b2, b0 ^ b3, b1);
//  - transposing 8-byte reads (4 consecutive rows r0..r0+3, r0 % 4 == 0, two adjacent chunk
//    columns c0, c0+1 with c0 even): positions (c0 ^ swz) and (c0 ^ swz ^ 1) over the four rows
//    are 8 distinct values because swz differs in bits 1-2 between rows with equal bits 2-3.
__device__ __forceinline__ int swz(int r) { return (((r & 3) << 1) | ((r >> 2) & 1)) ^ (((r >> 3) & 1) << 1); }

// Zero-fills rows row0 .. row0+nrows-1 (those below L) of a (row, head) slice [L][D]: the rows are
// contiguous in memory, so a wavefront writes 1 KB per instruction instead of 64 row pieces.
template <typename T>
__device__ __forceinline__ void zero_rows(T *head_ptr, int row0, int nrows, int L, int lane)
{
  char *base = reinterpret_cast<char *>(head_ptr + (size_t)row0 * D);
  const int bytes = max(0, min(nrows, L - row0)) * D * (int)sizeof(T);
  typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
  const u32x4_t z = {0u, 0u, 0u, 0u};
  for (int o = lane * 16; o < bytes; o += 1024) __builtin_nontemporal_store(z, reinterpret_cast<u32x4_t *>(base + o));
}

// Masks of a lane's 16 elements of a 32 x 32 accumulator tile, element i being row 4*half + 8*(i/4) + i%4 of the tile, as bits over
// the 32 rows: bits lo .. hi (any integers; hi < lo: none); and the elements of `x` whose bit is set, `other` in the place of the
// rest (of a NaN too).  Two vector instructions an element; a range test takes three and a scalar one.
__device__ __forceinline__ unsigned row_bits(int lo, int hi)
{
  const unsigned up_to = hi < 0 ? 0u : 0xFFFFFFFFu >> (31 - min(hi, 31));
  return lo > 31 ? 0u : up_to & (0xFFFFFFFFu << max(lo, 0));
}
__device__ __forceinline__ void keep_rows(f32x16 &x, unsigned bits, int half, float other = 0.0f)
{
  const int m = (int)(bits >> (4 * half));
  const unsigned rest = __float_as_uint(other);
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const unsigned keep = (unsigned)__builtin_amdgcn_sbfe(m, 8 * (i >> 2) + (i & 3), 1);
    x[i] = __uint_as_float((__float_as_uint(x[i]) & keep) | (rest & ~keep));
  }
}

// Two direct global->LDS loads of 16 bytes a lane, lane l's to lds + 16*l and 1 KB on, and the waits that go with them.  In assembly:
// of the compiler's own form it assumes that any LDS read may touch what is on its way, so a read from a buffer chosen at run time,
// and every __syncthreads(), waits for all of it, also for what was requested for later.  With these the kernel counts its
// outstanding requests itself: arrived_all<N>() returns when at most the last N of every wavefront of the workgroup are still on
// their way (and every wavefront's LDS reads so far are done).
// The destination is an operand in m0, which the compiler therefore sets and knows of (saved and put back by the assembly, which
// did as much for its safety: forward of the last position alone up to 0.7 % longer at B <= 9).  The second load's offset counts for both of
// its addresses, so the pair needs m0 once.
__device__ __forceinline__ unsigned lds_address(const void *p) { return (unsigned)(uintptr_t)(const lds_void *)p; }
constexpr int kLdsSlice = 1024;
// from base + off0, and from base + off1 + kLdsSlice
__device__ __forceinline__ void load_to_lds(const char *base, unsigned off0, unsigned off1, unsigned lds)
{
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %3\n\tglobal_load_lds_dwordx4 %2, %3 offset:%4" ::"{m0}"(lds), "v"(off0), "v"(off1),
               "s"(base), "n"(kLdsSlice)
               : "memory");
}
template <int N>
__device__ __forceinline__ void arrived_all()
{
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// two floats -> one register of two bf16 (round to nearest even in hardware: v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack2_bf16(float a, float b)
{
  const bf16x2 v = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(uint32_t, v);
}

// bf16 pair -> two floats and back (round to nearest even through the hardware conversion)
__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// x as hi + mid + lo with bf16 terms (exact for fp32 x), packed (hi | mid << 16, lo): the form
// in which one matrix instruction broadcasts a per-row constant into an accumulator
__device__ __forceinline__ uint2 split3(float x)
{
  const uint16_t hi = __builtin_bit_cast(uint16_t, (__bf16)x);
  const float r1 = x - bf16_to_f32(hi);
  const uint16_t mid = __builtin_bit_cast(uint16_t, (__bf16)r1);
  const uint16_t lo = __builtin_bit_cast(uint16_t, (__bf16)(r1 - bf16_to_f32(mid)));
  return make_uint2((uint32_t)hi | ((uint32_t)mid << 16), (uint32_t)lo);
}
__device__ __forceinline__ float unsplit3(uint32_t x, uint32_t y) { return (bf_lo(x) + bf_hi(x)) + bf_lo(y); }

// x as hi + lo with bf16 terms, packed hi | lo << 16
__device__ __forceinline__ uint32_t split2(float x)
{
  const uint16_t hi = __builtin_bit_cast(uint16_t, (__bf16)x);
  const uint16_t lo = __builtin_bit_cast(uint16_t, (__bf16)(x - bf16_to_f32(hi)));
  return (uint32_t)hi | ((uint32_t)lo << 16);
}
__device__ __forceinline__ float unsplit2(uint32_t x) { return bf_lo(x) + bf_hi(x); }

}  // namespace mfma
}  // namespace blossom
