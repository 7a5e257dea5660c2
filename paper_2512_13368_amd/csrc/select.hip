// Long-term block selection (Sec. 3.4): block compression (Eq. 9, phi = mean over the
// block's valid keys), importance scores (Eq. 10) and top-k (Eq. 13).
//
// The scores decide integers, so their arithmetic is fixed exactly: sequential fp32 sums in
// ascending position, one IEEE division, one fused-multiply-add chain over the channels.
// This file is compiled with -ffp-contract=off; the only fused operations are the explicit
// __fmaf_rn calls.  Plain ALUs only: the work is O(NB^2 d) per head and HBM-bound on the
// pooling pass.
#include <algorithm>

#include "common.h"
#include "launch.h"
#include "mfma_common.h"

namespace blossom {

// 16 bytes as floats.
__device__ __forceinline__ void unpack(const uint4 &v, float (&o)[4])
{
  o[0] = __uint_as_float(v.x); o[1] = __uint_as_float(v.y); o[2] = __uint_as_float(v.z); o[3] = __uint_as_float(v.w);
}
__device__ __forceinline__ void unpack(const uint4 &v, float (&o)[8])
{
  const unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    o[2 * i] = __uint_as_float(w[i] << 16);
    o[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
  }
}

__device__ __forceinline__ void unpack(const uint2 &v, float (&o)[4])
{
  o[0] = __uint_as_float(v.x << 16); o[1] = __uint_as_float(v.x & 0xFFFF0000u);
  o[2] = __uint_as_float(v.y << 16); o[3] = __uint_as_float(v.y & 0xFFFF0000u);
}

// Sum of a block's valid positions, in ascending order, for 16 bytes of channels of one tensor: kPoolBatch rows are in
// flight at a time (a rolled loop, which the compiler unrolled without hoisting a load, waited for each row in turn:
// the one-workgroup selection of B=128 H=4 L=1024 d=64 bf16 took 32 us, 24 now).  Rows past the end are read as the last one and add +0, which
// changes nothing: a sum that starts from +0 is never -0.
template <typename T, int D, int kPoolBatch, int EPT>
__device__ __forceinline__ void pool_batches(const T *__restrict__ src, int lo, int hi, float (&a)[EPT])
{
  for (int t = lo; t < hi; t += kPoolBatch) {
    using V = std::conditional_t<EPT * sizeof(T) == 16, uint4, uint2>;
    V v[kPoolBatch];
#pragma unroll
    for (int i = 0; i < kPoolBatch; ++i) v[i] = *reinterpret_cast<const V *>(src + (size_t)min(t + i, hi - 1) * D);
#pragma unroll
    for (int i = 0; i < kPoolBatch; ++i) {
      float x[EPT];
      unpack(v[i], x);
#pragma unroll
      for (int e = 0; e < EPT; ++e) a[e] = a[e] + (t + i < hi ? x[e] : 0.0f);
    }
  }
}

// The same for a whole number of pairs of eight rows: the next eight are requested before the last eight are added, and no row
// needs a test (pooling at B=16 H=8 L=8192 d=64 b=64: 55.6 -> 53.9 us, K alone 29.3 -> 27.8; where blocks of one wavefront
// differ in their valid rows, as in the selection of a whole head, both forms would run: 24 -> 29 us at L=1024).
template <bool STREAM, typename T, int D, int EPT>
__device__ __forceinline__ void pool_rows(const T *__restrict__ src, int n, float (&a)[EPT])
{
  using V = std::conditional_t<EPT * sizeof(T) == 16, uint4, uint2>;
  constexpr int R = 8;
  V u[R], v[R];
  auto request = [&](V (&x)[R], int t) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const V *row = reinterpret_cast<const V *>(src + (size_t)(t + i) * D);
      if constexpr (STREAM) x[i] = load_once(row);
      else x[i] = *row;
    }
  };
  auto add = [&](const V (&x)[R]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < R; ++i) {
      float f[EPT];
      unpack(x[i], f);
#pragma unroll
      for (int e = 0; e < EPT; ++e) a[e] = a[e] + f[e];
    }
  };
  request(u, 0);
  request(v, R);
  int t = 2 * R;
  for (; t < n; t += 2 * R) {
    add(u);
    request(u, t);
    add(v);
    request(v, t + R);
  }
  add(u);
  add(v);
}

template <typename T, int D, int EPT>
__device__ __forceinline__ void pool_block(const T *__restrict__ src, int lo, int hi, float (&a)[EPT])
{
#pragma unroll
  for (int e = 0; e < EPT; ++e) a[e] = 0.0f;
  if (hi - lo > 8) pool_batches<T, D, 16>(src, lo, hi, a);
  else pool_batches<T, D, 8>(src, lo, hi, a);
}

// Where the mean of channel c of key block J of head bh goes: rows of d channels, or transposed, for the scoring with a thread per
// candidate: beyond kRowBlocks blocks, and for the last block alone beyond half of that (selection + forward at d=64 b=64 L=6000, us, with
// rows and transposed: B=1 H=8 25.1 / 24.6, B=5 28.0 / 27.2, B=12 36.3 / 36.0; with 63 blocks, B=12 H=8 L=2000 b=32, 28.2 / 28.7).
constexpr int kRowBlocks = 128;
__host__ __device__ __forceinline__ bool means_in_rows(const KParams &p) { return p.NB <= (p.nq == 1 ? kRowBlocks / 2 : kRowBlocks); }
template <int D>
__device__ __forceinline__ size_t kmean_at(int bh, int J, int c, const KParams &p)
{
  return means_in_rows(p) ? ((size_t)bh * p.NB + J) * D + c : ((size_t)bh * D + c) * p.NB + J;
}

// ---- pooling ------------------------------------------------------------------------------
// One lane owns 16 bytes of channels of one block of one tensor.  qsum [B,H,NB,d] (unnormalised sums of Q), kmean: above.
// KCMP: K holds compressed keys [B,H,NB,d] supplied by the caller (Eq. 9 with the caller's phi);
// they are copied as they are instead of being pooled.
// STREAM: whole blocks are read past the caches (see kKeysOnceBytes).
template <typename T, int D, bool KCMP, bool STREAM>
__global__ __launch_bounds__(256) void pool_kernel(const T *__restrict__ Q, const T *__restrict__ K,
                                                   const int *__restrict__ valid_len,
                                                   float *__restrict__ qsum, float *__restrict__ kmean,
                                                   KParams p)
{
  constexpr int EPT = 4;
  constexpr int LPT = D / EPT;  // lanes per (tensor, row-head, block) task
  const long n_bhj = (long)p.B * p.H * p.NB;
  const long task = (long)blockIdx.x * (256 / LPT) + threadIdx.x / LPT;
  if (task >= 2 * n_bhj) return;
  const int c0 = (threadIdx.x % LPT) * EPT;
  const int which = task >= n_bhj;
  const long rem = which ? task - n_bhj : task;
  const int bh = (int)(rem / p.NB);
  const int J = (int)(rem % p.NB);
  if (!which && J < p.NB - p.nq) return;  // serving mode: only the last query block is pooled
  float a[EPT];
  if (KCMP && which) {
#pragma unroll
    for (int e = 0; e < EPT; e += 4) load4(K + ((size_t)bh * p.NB + J) * D + c0 + e, reinterpret_cast<float(&)[4]>(a[e]));
#pragma unroll
    for (int e = 0; e < EPT; ++e) kmean[kmean_at<D>(bh, J, c0 + e, p)] = a[e];
    return;
  }
  const int p0 = p.L - clamp_len(valid_len[bh / p.H], p.L);
  const int lo = max(J * p.b, p0), hi = min((J + 1) * p.b, p.L);
  const T *src = (which ? K : Q) + (size_t)bh * p.L * D + c0;
  // (A ragged block among a wavefront's whole ones makes it run both loops, worth it while that block is a quarter of one at most:
  // selection with d=64 b=64, us, both loops and one for all, B=4 H=4 L=5105, 49 rows left over, 12.2 / 11.0; B=9 H=4 L=3396, 4 rows,
  // 10.5 / 12.2; B=2 H=4 L=2637, 13 rows, 9.4 / 9.8; with b=32 B=1 H=8 L=1242, 26 rows, 9.2 / 8.5.)
  if (p.b >= 32 && __all(hi - lo == p.b || hi - lo <= p.b / 4) && hi - lo == p.b) {
#pragma unroll
    for (int e = 0; e < EPT; ++e) a[e] = 0.0f;
    pool_rows<STREAM, T, D>(src + (size_t)lo * D, p.b, a);
  } else {
    pool_block<T, D, EPT>(src, lo, hi, a);
  }
  if (!which) {
#pragma unroll
    for (int e = 0; e < EPT; e += 4)
      store4(qsum + ((size_t)bh * p.NB + J) * D + c0 + e, reinterpret_cast<float(&)[4]>(a[e]));
  } else {
    const float fc = (float)(hi - lo);
#pragma unroll
    for (int e = 0; e < EPT; ++e)
      kmean[kmean_at<D>(bh, J, c0 + e, p)] = hi > lo ? __fdiv_rn(a[e], fc) : 0.0f;
  }
}

// ---- pooling with the rotary position embedding applied on the way in (Sec. 3.3) ------------
// Every position (padding too) is rotated with the caller's cos/sin tables, rounded to the storage
// type and written to Q_rot / K_rot; the pooled sums are taken over those rounded values, so that
// selection, forward and backward all see the same rotated tensors.  Fixed fp32 recipe on channel
// pairs (2i, 2i+1) at position m: t = x1*s; x0' = fma(x0, c, -t); u = x1*c; x1' = fma(x0, s, u).
//
// One workgroup per (tensor, row-head, run of kRopeRows positions): the run is one contiguous chunk
// of memory, read and written with 16 bytes per lane, consecutive lanes on consecutive addresses.
// The rotated values also go to LDS (fp32), from where one thread per (block of the run, channel)
// takes the block's sum in ascending position order.
constexpr int kRopeRows = 64;

template <typename T, int D>
__global__ __launch_bounds__(256) void rope_pool_kernel(const T *__restrict__ Q, const T *__restrict__ K,
                                                        const int *__restrict__ valid_len,
                                                        float *__restrict__ qsum, float *__restrict__ kmean,
                                                        T *__restrict__ Q_rot, T *__restrict__ K_rot, KParams p)
{
  constexpr int EPT = 16 / (int)sizeof(T);  // elements of a 16-byte piece: 8 bf16 or 4 fp32
  constexpr int PPR = D / EPT;              // pieces per row
  __shared__ __attribute__((aligned(16))) float rot_s[kRopeRows][D];  // (rows are read with one channel per lane: no padding needed)
  const int runs = (p.L + kRopeRows - 1) / kRopeRows;
  const int BH = p.B * p.H;
  const int which = blockIdx.x >= (unsigned)(BH * runs);
  const int rem = (int)blockIdx.x - which * BH * runs;
  const int bh = rem / runs, run = rem % runs;
  const int t_lo = run * kRopeRows, t_hi = min(t_lo + kRopeRows, p.L);
  const int J_lo = t_lo / p.b, J_hi = (t_hi - 1) / p.b;  // blocks of the run (kRopeRows is a multiple of every b)
  if (!which && J_hi < p.NB - p.nq) return;              // serving mode: queries of the last block only
  const T *src = (which ? K : Q) + ((size_t)bh * p.L + t_lo) * D;
  T *dst = (which ? K_rot : Q_rot) + ((size_t)bh * p.L + t_lo) * D;
  const int pieces = (t_hi - t_lo) * PPR;
  for (int q = threadIdx.x; q < pieces; q += 256) {
    const int r = q / PPR, c0 = (q % PPR) * EPT;
    const int t = t_lo + r;
    float x[EPT], y[EPT], cs[EPT / 2], sn[EPT / 2];
    if constexpr (EPT == 8) {
      load4(src + (size_t)q * EPT, reinterpret_cast<float(&)[4]>(x[0]));
      load4(src + (size_t)q * EPT + 4, reinterpret_cast<float(&)[4]>(x[4]));
      const float4 c = *reinterpret_cast<const float4 *>(p.rope_cos + (size_t)t * (D / 2) + c0 / 2);
      const float4 s4 = *reinterpret_cast<const float4 *>(p.rope_sin + (size_t)t * (D / 2) + c0 / 2);
      cs[0] = c.x; cs[1] = c.y; cs[2] = c.z; cs[3] = c.w;
      sn[0] = s4.x; sn[1] = s4.y; sn[2] = s4.z; sn[3] = s4.w;
    } else {
      load4(src + (size_t)q * EPT, reinterpret_cast<float(&)[4]>(x[0]));
      const float2 c = *reinterpret_cast<const float2 *>(p.rope_cos + (size_t)t * (D / 2) + c0 / 2);
      const float2 s2 = *reinterpret_cast<const float2 *>(p.rope_sin + (size_t)t * (D / 2) + c0 / 2);
      cs[0] = c.x; cs[1] = c.y;
      sn[0] = s2.x; sn[1] = s2.y;
    }
#pragma unroll
    for (int i = 0; i < EPT / 2; ++i) {
      y[2 * i] = __fmaf_rn(x[2 * i], cs[i], -__fmul_rn(x[2 * i + 1], sn[i]));
      y[2 * i + 1] = __fmaf_rn(x[2 * i], sn[i], __fmul_rn(x[2 * i + 1], cs[i]));
    }
#pragma unroll
    for (int e = 0; e < EPT; ++e) y[e] = to_f32(from_f32<T>(y[e]));  // what the attention kernels will read
#pragma unroll
    for (int e = 0; e < EPT; e += 4)
      *reinterpret_cast<float4 *>(&rot_s[r][c0 + e]) = make_float4(y[e], y[e + 1], y[e + 2], y[e + 3]);
    store4(dst + (size_t)q * EPT, reinterpret_cast<float(&)[4]>(y[0]));
    if constexpr (EPT == 8) store4(dst + (size_t)q * EPT + 4, reinterpret_cast<float(&)[4]>(y[4]));
  }
  __syncthreads();
  const int p0 = p.L - clamp_len(valid_len[bh / p.H], p.L);
  const int nblk = J_hi - J_lo + 1;
  for (int e = threadIdx.x; e < nblk * D; e += 256) {
    const int J = J_lo + e / D, c = e % D;
    if (!which && J < p.NB - p.nq) continue;
    const int lo = max(J * p.b, p0), hi = min((J + 1) * p.b, p.L);
    float a = 0.0f;
#pragma unroll 8
    for (int t = lo; t < hi; ++t) a = a + rot_s[t - t_lo][c];
    if (!which) {
      qsum[((size_t)bh * p.NB + J) * D + c] = a;
    } else {
      const int cnt = hi - lo;
      kmean[kmean_at<D>(bh, J, c, p)] = cnt > 0 ? __fdiv_rn(a, (float)cnt) : 0.0f;
    }
  }
}

// ---- scoring + top-k ----------------------------------------------------------------------
// Each score becomes an order-preserving integer image of the fp32 value (with -0 folded onto +0, so that equal
// scores give equal images); "beats" under (score descending, index ascending) compares the images, then the indexes.
// In the bidirectional form the query's own block is a candidate with the largest possible image: it is always taken
// and comes out at its place in the ascending list.  In the causal form it closes the list.
__device__ __forceinline__ unsigned score_image(float score)
{
  unsigned u = __float_as_uint(score);
  if (u == 0x80000000u) u = 0u;                    // -0 ties with +0
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);  // monotone in the score
}

// The candidates of query block I of a row whose valid positions start at p0: [J_first, J_end), and how many are taken.
struct Candidates {
  int J_first, J_end, take;
  bool any;  // the block holds a valid query
};
__device__ __forceinline__ Candidates candidates(const KParams &p, int p0, int I)
{
  Candidates c;
  c.any = min((I + 1) * p.b, p.L) > p0;
  c.J_first = p0 / p.b;
  c.J_end = p.bidir ? p.NB : I;
  const int n_cand = p.bidir ? p.NB - c.J_first - 1 : I - c.J_first;
  c.take = min(p.k - 1, n_cand) + (p.bidir ? 1 : 0);
  if (!c.any) c.take = 0;
  return c;
}

// One fused-multiply-add chain over the channels, in ascending order; rows of d floats in LDS.
template <int D>
__device__ __forceinline__ float score_dot(const float *q, const float *k)
{
  float acc = 0.0f;
#pragma unroll
  for (int c = 0; c < D; c += 4) {
    const float4 a = *reinterpret_cast<const float4 *>(q + c), b = *reinterpret_cast<const float4 *>(k + c);
    acc = __fmaf_rn(a.x, b.x, acc);
    acc = __fmaf_rn(a.y, b.y, acc);
    acc = __fmaf_rn(a.z, b.z, acc);
    acc = __fmaf_rn(a.w, b.w, acc);
  }
  return acc;
}

// Up to 32 blocks: one thread per (query block, candidate) pair.  A candidate is selected iff fewer than `take` beat it;
// a query block's choices are the bits of one word, written out with consecutive threads on consecutive entries.
// scratch: NB*NB images, then NB words.  Every thread of the workgroup calls it, after a barrier.
constexpr int kPairBlocks = 32;
template <int D>
__device__ void pick_by_pairs(const float *q_s, const float *k_s, unsigned *scratch, int *__restrict__ out, int p0,
                              const KParams &p)
{
  const int tid = threadIdx.x, nt = blockDim.x, NB = p.NB, I0 = NB - p.nq;
  unsigned *img = scratch, *chosen = scratch + NB * NB;
  // causal: rows I and NB-1-I together hold NB-1 candidates
  const int pairs = p.bidir ? NB * NB : (NB + 1) / 2 * (NB - 1);
  auto pair = [&](int e, int &I, int &J) {
    const int w = p.bidir ? NB : NB - 1, r = e / w, c = e - r * w;
    I = r;
    J = c;
    if (!p.bidir) {
      const int big = NB - 1 - r;
      I = c < big ? big : r;
      J = c < big ? c : c - big;
      if (c >= big && big == r) return false;  // the middle row of an odd count stands alone
    }
    return I >= I0 && J >= p0 / p.b;
  };
  for (int I = tid; I < NB; I += nt) {
    const Candidates c = candidates(p, p0, I);
    chosen[I] = c.any && !p.bidir ? 1u << I : 0u;
  }
  for (int e = tid; e < pairs; e += nt) {
    int I, J;
    if (!pair(e, I, J)) continue;
    img[I * NB + J] = p.bidir && I == J ? ~0u : score_image(score_dot<D>(q_s + (I - I0) * (D + 4), k_s + J * (D + 4)));
  }
  __syncthreads();
  for (int e = tid; e < pairs; e += nt) {
    int I, J;
    if (!pair(e, I, J)) continue;
    const Candidates c = candidates(p, p0, I);
    const unsigned mine = img[I * NB + J];
    int rank = 0;
    for (int Jo = c.J_first; Jo < c.J_end; ++Jo) {
      const unsigned other = img[I * NB + Jo];
      rank += other > mine || (other == mine && Jo < J) ? 1 : 0;
    }
    if (rank < c.take) atomicOr(&chosen[I], 1u << J);
  }
  __syncthreads();
  for (int e = tid; e < p.nq * p.k; e += nt) {
    const int r = e / p.k;
    unsigned m = chosen[I0 + r];
    for (int slot = e - r * p.k; slot > 0 && m; --slot) m &= m - 1;
    out[(size_t)I0 * p.k + e] = m ? __builtin_ctz(m) : -1;
  }
}

// Up to 128 blocks: a wavefront takes kRowsPerWave query blocks at a time, one or two candidates per lane.  The query rows
// lie across the lanes too and are read channel by channel into scalar registers.  The take-th largest image of a row is
// found bit by bit from the top (a compare and a population count per bit and slot: the scalar unit does most of it, and
// a vector instruction costs four cycles), the rows' searches independent of each other and given up as soon as exactly
// `take` images are left above the line.  (Ranks by counting the larger images, as for the pairs: 17 against 15 us at
// B=32 H=8 L=1997 d=64, 63 blocks.)
// q(r): the row r's channel `lane` (any value from lane d on).
constexpr int kRowsPerWave = 4;
__device__ __forceinline__ float lane_value(float v, int lane)
{
  return __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)__float_as_uint(v), lane));
}
// Few picks (the paper's three): the largest image is taken as often, with all that equal it.  Its cost goes with the passes (one more in
// the bidirectional form, where the own block is a candidate), the search's with how far apart the images lie.  Selection alone,
// us, passes against search: three passes at B=32 H=8 L=2000 d=8 14.6 / 20.9, L=1997 d=64 b=32 25.6 / 26.8; five 16.8 / 20.0 and 26.6 / 26.8,
// bidirectional at B=128 H=8 L=1024 d=64 b=16 68.6 / 69.8; six 17.8 / 20.2 and 27.1 / 26.9, 70.0 / 70.2; seven 18.9 / 20.1 and 27.5 / 27.4,
// 71.6 / 70.3.
constexpr int kFewPasses = 5;
// the largest over the wavefront, in a scalar register: inside rows of 16 lanes, then the four rows
__device__ __forceinline__ unsigned lanes_max(unsigned x)
{
  x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xf, 0xf, false));
  x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xf, 0xf, false));
  x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xf, 0xf, false));
  x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x140, 0xf, 0xf, false));
  auto row = [&](int i) { return (unsigned)__builtin_amdgcn_readlane((int)x, 16 * i); };
  return max(max(row(0), row(1)), max(row(2), row(3)));
}
template <int D, int SLOTS, int R, typename QRow>
__device__ __forceinline__ void pick_rows(QRow &&q, const float *k_s, int *__restrict__ out, int I0, int I1, int p0,
                                          const KParams &p)
{
  const int lane = threadIdx.x & 63;
  const int J_first = p0 / p.b;
  int J[SLOTS];
  const float *k[SLOTS];
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    J[s] = J_first + lane + 64 * s;
    k[s] = k_s + min(J[s], p.NB - 1) * (D + 4);
  }
  float acc[R][SLOTS], qv[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    qv[r] = q(min(r, I1 - 1 - I0));
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) acc[r][s] = 0.0f;
  }
#pragma unroll 4
  for (int c0 = 0; c0 < D; c0 += 4) {
    float kv[SLOTS][4];
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) load4(k[s] + c0, kv[s]);
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const float qc = lane_value(qv[r], c0 + c);
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) acc[r][s] = __fmaf_rn(qc, kv[s][c], acc[r][s]);
      }
  }
  unsigned u[R][SLOTS], line[R];  // images: 0, below every other, where there is no candidate
  int take[R], above[R];          // above: images at or above the line
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const Candidates c = candidates(p, p0, I0 + r);
    take[r] = c.take;
    above[r] = -1;
    line[r] = 0u;
#pragma unroll
    for (int s = 0; s < SLOTS; ++s)
      u[r][s] = J[s] >= c.J_end ? 0u : p.bidir && J[s] == I0 + r ? ~0u : score_image(acc[r][s]);
  }
  if (p.k - 1 + p.bidir <= kFewPasses) {
    unsigned v[R][SLOTS];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      above[r] = 0;
#pragma unroll
      for (int s = 0; s < SLOTS; ++s) v[r][s] = u[r][s];
    }
    for (bool done = false; !done;) {
      done = true;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        unsigned m = v[r][0];
#pragma unroll
        for (int s = 1; s < SLOTS; ++s) m = max(m, v[r][s]);
        m = lanes_max(m);
        int cnt = 0;
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
          cnt += __popcll(__ballot(v[r][s] == m));
          v[r][s] = v[r][s] == m ? 0u : v[r][s];
        }
        line[r] = above[r] < take[r] ? m : line[r];
        above[r] += cnt;
        done = done && above[r] >= take[r];
      }
    }
  } else {
    for (int bit = 31; bit >= 0; --bit) {
      bool done = true;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const unsigned test = line[r] | (1u << bit);
        int cnt = 0;
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) cnt += __popcll(__ballot(u[r][s] >= test));
        line[r] = cnt >= take[r] ? test : line[r];
        above[r] = cnt >= take[r] ? cnt : above[r];
        done = done && above[r] == take[r];
      }
      if (done) break;
    }
  }
  const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int I = I0 + r;
    if (I >= I1) break;
    unsigned long long ch[SLOTS], eq[SLOTS];
    int left = take[r];
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
      ch[s] = take[r] > 0 ? __ballot(u[r][s] > line[r]) : 0ull;
      eq[s] = __ballot(u[r][s] == line[r]);
      left -= __popcll(ch[s]);
    }
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {  // of the images on the line, the first `left` in ascending block order
      ch[s] |= __ballot(((eq[s] >> lane) & 1ull) && (int)__popcll(eq[s] & below) < left);
      left -= __popcll(eq[s]);
    }
    int *row = out + (size_t)I * p.k;
    int base = 0;
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
      if ((ch[s] >> lane) & 1ull) row[base + __popcll(ch[s] & below)] = J[s];
      base += __popcll(ch[s]);
    }
    if (!p.bidir && candidates(p, p0, I).any) {
      if (lane == 0) row[base] = I;
      ++base;
    }
    for (int e = base + lane; e < p.k; e += 64) row[e] = -1;
  }
}
template <int D>
__device__ __forceinline__ void pick_by_rows(const float *q_s, const float *k_s, int *__restrict__ out, int I0, int I1, int p0,
                                             const KParams &p)
{
  const int waves = blockDim.x >> 6, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  auto go = [&](auto rows) {
    constexpr int R = decltype(rows)::value;
    for (int I = I0 + R * wave; I < I1; I += R * waves) {
      const int last = min(I + R, I1);
      auto q = [&](int r) { return q_s[(I - I0 + r) * (D + 4) + (threadIdx.x & (D - 1))]; };
      if ((p.bidir ? p.NB : last - 1) - p0 / p.b > 64) pick_rows<D, 2, R>(q, k_s, out, I, last, p0, p);
      else pick_rows<D, 1, R>(q, k_s, out, I, last, p0, p);
    }
  };
  if (I1 - I0 <= waves) go(std::integral_constant<int, 1>{});  // (serving mode: one row)
  else go(std::integral_constant<int, kRowsPerWave>{});
}

// LDS of a workgroup that scores `rows` query blocks of a head: padded rows of d + 4 floats, and the pairs' images.
static size_t pick_lds(const KParams &p, int rows)
{
  const size_t pairs = p.NB <= kPairBlocks ? (size_t)p.NB * p.NB + p.NB : 0;
  return ((size_t)(rows + p.NB) * (p.d + 4) + pairs) * sizeof(float);
}

// Pooling, scoring and top-k of one head in one workgroup: the pooled rows stay in LDS.  As two kernels the
// pooled rows went through memory, and the second, a wavefront per query block, was all latency: at
// B=2048 H=8 L=200 d=16 fp32 it took 55 us after 58 us of pooling, at B=128 H=4 L=1024 d=64 bf16 15 after 25.
template <typename T, int D>
__global__ __launch_bounds__(1024) void select_head_kernel(const T *__restrict__ Q, const T *__restrict__ K,
                                                           const int *__restrict__ valid_len, int *__restrict__ sel, KParams p)
{
  constexpr int EPT = 16 / (int)sizeof(T);
  constexpr int LPT = D / EPT;
  extern __shared__ __attribute__((aligned(16))) float sel_lds[];
  float *q_s = sel_lds, *k_s = q_s + p.nq * (D + 4);
  const int bh = blockIdx.x;
  const int p0 = p.L - clamp_len(valid_len[bh / p.H], p.L);
  for (int e = threadIdx.x; e < (p.nq + p.NB) * LPT; e += blockDim.x) {
    const int row = e / LPT, c0 = (e % LPT) * EPT;
    const bool key = row >= p.nq;
    const int J = key ? row - p.nq : p.NB - p.nq + row;
    const int lo = max(J * p.b, p0), hi = min((J + 1) * p.b, p.L);
    float a[EPT];
    pool_block<T, D, EPT>((key ? K : Q) + (size_t)bh * p.L * D + c0, lo, hi, a);
    if (key) {
      const float fc = (float)(hi - lo);
#pragma unroll
      for (int i = 0; i < EPT; ++i) a[i] = hi > lo ? __fdiv_rn(a[i], fc) : 0.0f;
    }
#pragma unroll
    for (int i = 0; i < EPT; i += 4) store4(q_s + row * (D + 4) + c0 + i, reinterpret_cast<float(&)[4]>(a[i]));
  }
  __syncthreads();
  int *out = sel + (size_t)bh * p.NB * p.k;
  if (p.NB <= kPairBlocks)
    pick_by_pairs<D>(q_s, k_s, reinterpret_cast<unsigned *>(k_s + p.NB * (D + 4)), out, p0, p);
  else
    pick_by_rows<D>(q_s, k_s, out, p.NB - p.nq, p.NB, p0, p);
}

// Scoring and top-k of pooled rows, means in rows: a workgroup per kScoreRows query blocks of a head (or per head,
// where the pairs do it), which holds the head's key means in LDS.
constexpr int kScoreRows = 16;
template <int D>
__global__ __launch_bounds__(256) void score_topk_kernel(const float *__restrict__ qsum, const float *__restrict__ kmean,
                                                         const int *__restrict__ valid_len, int *__restrict__ sel, int rows,
                                                         KParams p)
{
  extern __shared__ __attribute__((aligned(16))) float sel_lds[];
  const int chunks = (p.nq + rows - 1) / rows;
  // (a head's chunks on one XCD, which has the means in its L2; in turn they would give one XCD the last, longest chunks of all)
  const unsigned vid = mfma::xcd_spread(blockIdx.x, gridDim.x / chunks, chunks);
  const int bh = (int)(vid / chunks);
  const int I0 = p.NB - p.nq + (int)(vid % chunks) * rows, I1 = min(I0 + rows, p.NB);
  float *q_s = sel_lds, *k_s = q_s + rows * (D + 4);
  const int p0 = p.L - clamp_len(valid_len[bh / p.H], p.L);
  auto stage = [&](float *to, const float *from, int lo, int hi) {  // eight loads in flight per thread
    const int end = hi * (D / 4);
    for (int e0 = lo * (D / 4) + (int)threadIdx.x; e0 < end; e0 += 8 * 256) {
      float4 v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = reinterpret_cast<const float4 *>(from)[min(e0 + i * 256, end - 1)];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int e = e0 + i * 256;
        if (e < end) *reinterpret_cast<float4 *>(to + e / (D / 4) * (D + 4) + e % (D / 4) * 4) = v[i];
      }
    }
  };
  stage(q_s, qsum + ((size_t)bh * p.NB + I0) * D, 0, I1 - I0);
  stage(k_s, kmean + (size_t)bh * p.NB * D, p0 / p.b, p.bidir ? p.NB : I1);  // (I1 <= NB)
  __syncthreads();
  int *out = sel + (size_t)bh * p.NB * p.k;
  if (p.NB <= kPairBlocks)
    pick_by_pairs<D>(q_s, k_s, reinterpret_cast<unsigned *>(k_s + p.NB * (D + 4)), out, p0, p);
  else
    pick_by_rows<D>(q_s, k_s, out, I0, I1, p0, p);
}

// Means stored transposed (means_in_rows): a workgroup per (row, head, query block), thread-strided candidates, keys (the image above
// NB-1-J: unique, one unsigned comparison) in LDS.  A candidate is selected iff fewer than `take` candidates beat it;
// ballots and prefix popcounts emit the list in ascending order.
// Latency is the bound, so a candidate has a thread of its own, 32 of its channels are requested before the first is used, and the
// ranks are counted without a wait.  Selection at d=64 b=32 L=8192, 256 blocks, with a wavefront per row, the same with these requests,
// and with these threads, us: the last block alone at B=16 H=8 84 / 54 / 39, at B=1 H=8 59 / 27 / 12; every block at B=1 H=8
// 61 / 32 / 26, B=4 92 / 87 / 54, B=16 204 / 191 / 182.
template <int D>
__global__ __launch_bounds__(1024) void score_topk_many_kernel(const float *__restrict__ qsum,
                                                               const float *__restrict__ kmeanT,
                                                               const int *__restrict__ valid_len,
                                                               int *__restrict__ sel, KParams p)
{
  __shared__ __attribute__((aligned(16))) float qs[D];
  __shared__ unsigned long long chosen_s[64];   // per 64 candidates (NB <= 4096)
  extern __shared__ unsigned long long key_s[];  // NB keys (sized at launch: a static worst-case array would cap the occupancy)
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63;
  const int I = p.NB - p.nq + (int)(blockIdx.x % p.nq);
  const int bh = blockIdx.x / p.nq;
  const int p0 = p.L - clamp_len(valid_len[bh / p.H], p.L);
  int *out = sel + ((size_t)bh * p.NB + I) * p.k;
  const Candidates cd = candidates(p, p0, I);
  if (!cd.any) {
    for (int e = tid; e < p.k; e += nt) out[e] = -1;
    return;
  }
  for (int c = tid; c < D; c += nt) qs[c] = qsum[((size_t)bh * p.NB + I) * D + c];
  __syncthreads();
  const float *km = kmeanT + (size_t)bh * D * p.NB;
  for (int J = cd.J_first + tid; J < cd.J_end; J += nt) {
    constexpr int R = D < 32 ? D : 32;  // channels on their way at a time
    const float *from = km + J;
    float acc = 0.0f;
#pragma unroll 1
    for (int c0 = 0; c0 < D; c0 += R) {
      float v[R];
#pragma unroll
      for (int c = 0; c < R; ++c, from += p.NB) v[c] = *from;
#pragma unroll
      for (int c = 0; c < R; ++c) acc = __fmaf_rn(qs[c0 + c], v[c], acc);
    }
    key_s[J] = J == I ? ~0ull : ((unsigned long long)score_image(acc) << 32) | (unsigned)(p.NB - 1 - J);
  }
  __syncthreads();
  auto below = [&](unsigned long long m) { return __popcll(m & ((1ull << lane) - 1ull)); };
  for (int J0 = cd.J_first + (tid & ~63); J0 < cd.J_end; J0 += nt) {
    const int J = J0 + lane;
    int rank = cd.take;
    if (J < cd.J_end) {
      const unsigned long long mine = key_s[J];
      rank = 0;
#pragma unroll 8
      for (int Jo = cd.J_first; Jo < cd.J_end; ++Jo) rank += key_s[Jo] > mine ? 1 : 0;
    }
    const unsigned long long mask = __ballot(rank < cd.take);
    if (lane == 0) chosen_s[(J0 - cd.J_first) >> 6] = mask;
  }
  __syncthreads();
  for (int J0 = cd.J_first + (tid & ~63); J0 < cd.J_end; J0 += nt) {
    const int c = (J0 - cd.J_first) >> 6;
    int base = 0;
    for (int o = 0; o < c; ++o) base += __popcll(chosen_s[o]);
    const unsigned long long mask = chosen_s[c];
    if ((mask >> lane) & 1ull) out[base + below(mask)] = J0 + lane;
  }
  // `take` are selected; causal form: the own block closes the list; the rest is padding
  if (!p.bidir && tid == 0) out[cd.take] = I;
  for (int e = cd.take + (p.bidir ? 0 : 1) + tid; e < p.k; e += nt) out[e] = -1;
}

// ---- launchers ----------------------------------------------------------------------------
// One workgroup per head pools the whole of it, up to kHeadBytes of Q and K (beyond, the longest row of a batch sets the
// time, not the memory).  With more than 32 blocks the scoring is no longer short, and fewer than kHeads heads leave CUs
// idle through it: at B=30 H=8 L=2000 d=64 b=32 one workgroup per head takes 23 us and two kernels 29, at B=8 18 and 14.
constexpr size_t kHeadBytes = 512 * 1024;
constexpr long kHeads = 192;
static bool one_workgroup_per_head(const KParams &p, size_t elem)
{
  if ((size_t)(p.L + std::min(p.L, p.nq * p.b)) * p.d * elem > kHeadBytes) return false;
  if (p.NB > kRowBlocks || pick_lds(p, p.nq) > 64 * 1024) return false;
  return p.NB <= kPairBlocks || (long)p.B * p.H >= kHeads;
}

// Keys of the last block's selection are read past the caches where there are many: nothing reads most of them again, and pooling at
// B=16 H=8 L=8192 d=64 b=64 takes 24 instead of 27 us.  Fewer may be in the last-level cache (256 MB), from whoever made them, and those of
// a whole selection are read again by the forward (B=700 H=8 L=200 d=16 fp32, 143 MB, 111.7 us without and 115.0 with).  Selection +
// forward of the last block, H=8 d=64 b=64 bf16, through / past the caches, us, with other keys than the last call's, and (a copy of
// them in both figures) with keys written right before the call:
//   64 MB  B=16 H=4 L=8192  37.2 / 37.9    64.4 / 65.7       101 MB  B=16 L=6500  46.4 / 44.9   83.9 / 83.6
//   70 MB  B=16 L=4500      38.7 / 38.6    66.4 / 66.4       117 MB  B=16 L=7500  48.7 / 47.2   92.4 / 92.0
//   85 MB  B=16 L=5500      43.7 / 42.7    76.2 / 75.8       128 MB  B=16 L=8192  52.4 / 49.4   98.6 / 97.9
//   96 MB  B=12 L=8192      45.6 / 44.0    81.4 / 82.2       256 MB  B=32 L=8192  80.5 / 74.9    188 / 171
// The line lies where both gain.  (The same keys in one call after another: 101 MB 41.9 / 44.9, 256 MB 71.9 / 74.6, 512 MB 145 / 131.)
constexpr size_t kKeysOnceBytes = 100u << 20;
template <typename T, int D>
static void launch_select_t(const KParams &p, const void *Q, const void *K, bool kcmp, const int *valid_len,
                            int *sel, void *ws, void *Q_rot, void *K_rot, hipStream_t st)
{
  constexpr int LPT = D * (int)sizeof(T) / 16;  // (select_head_kernel's lanes per block)
  if (!kcmp && !p.rope_cos && one_workgroup_per_head(p, sizeof(T))) {
    const int lanes = std::max((p.nq + p.NB) * LPT, p.NB > kPairBlocks ? 64 * p.nq / kRowsPerWave : 0);
    const int threads = std::min(1024, (lanes + 63) / 64 * 64);
    hipLaunchKernelGGL((select_head_kernel<T, D>), dim3((unsigned)(p.B * p.H)), dim3((unsigned)threads), pick_lds(p, p.nq), st,
                       (const T *)Q, (const T *)K, valid_len, sel, p);
    return;
  }
  float *qsum = reinterpret_cast<float *>(ws);
  float *kmean = qsum + (size_t)p.B * p.H * p.NB * D;
  const long tasks = 2L * p.B * p.H * p.NB;
  const int per_wg = 256 / (D / 4);
  const unsigned grid = (unsigned)((tasks + per_wg - 1) / per_wg);
  if (kcmp) {
    BLOSSOM_LAUNCH((pool_kernel<T, D, true, false>), dim3(grid), dim3(256), 0, st, (const T *)Q, (const T *)K,
                   valid_len, qsum, kmean, p);
  } else if (p.rope_cos) {
    const long rgrid = 2L * p.B * p.H * ((p.L + kRopeRows - 1) / kRopeRows);
    BLOSSOM_LAUNCH((rope_pool_kernel<T, D>), dim3((unsigned)rgrid), dim3(256), 0, st,
                   (const T *)Q, (const T *)K, valid_len, qsum, kmean, (T *)Q_rot, (T *)K_rot, p);
  } else {
    auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, st, (const T *)Q, (const T *)K, valid_len, qsum, kmean, p);
    };
    const bool stream = p.nq == 1 && (size_t)p.B * p.H * p.L * D * sizeof(T) >= kKeysOnceBytes;
    stream ? go(pool_kernel<T, D, false, true>) : go(pool_kernel<T, D, false, false>);
    if (launch_failed()) return;
  }
  if (!means_in_rows(p)) {
    const int threads = std::min(1024, (p.NB + 63) / 64 * 64);
    hipLaunchKernelGGL((score_topk_many_kernel<D>), dim3((unsigned)(p.B * p.H * p.nq)), dim3((unsigned)threads),
                       (size_t)p.NB * sizeof(unsigned long long), st, qsum, kmean, valid_len, sel, p);
    return;
  }
  const int few = (long)p.B * p.H * p.nq < 1024L * kScoreRows ? 4 : kScoreRows;  // (1024 workgroups: four per CU)
  const int rows = p.NB <= kPairBlocks ? p.nq : std::min(p.nq, few);
  hipLaunchKernelGGL((score_topk_kernel<D>), dim3((unsigned)(p.B * p.H * ((p.nq + rows - 1) / rows))), dim3(256),
                     pick_lds(p, rows), st, qsum, kmean, valid_len, sel, rows, p);
}

size_t select_workspace_bytes(const KParams &p) { return 2 * (size_t)p.B * p.H * p.NB * p.d * sizeof(float); }

void launch_select(const KParams &p, int dtype, const void *Q, const void *K, bool kcmp, const int *valid_len,
                   int *sel, void *ws, hipStream_t st, void *Q_rot, void *K_rot)
{
  with_head_dim(p.d, [&](auto dim) {
    constexpr int D = decltype(dim)::value;
    if (dtype == 0) launch_select_t<float, D>(p, Q, K, kcmp, valid_len, sel, ws, Q_rot, K_rot, st);
    else launch_select_t<bf16_t, D>(p, Q, K, kcmp, valid_len, sel, ws, Q_rot, K_rot, st);
  });
}

}  // namespace blossom
