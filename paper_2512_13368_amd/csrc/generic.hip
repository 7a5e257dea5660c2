// Scalar-ALU kernels of the fused attention path for every supported (dtype, d, b):
// forward (both branches + gate, Eq. 1, 16-19), dense causal comparison, and the backward
// pass (gate backward, dQ, inverse selection list, dK/dV, gate-gradient reduction).
//
// Lane mapping: one wavefront per (row, head, block).  A lane owns one row of the block and
// one "phase" of the key (or query) tile: with block size b there are 64/b phases, each
// walking every (64/b)-th row of a tile staged in LDS with its own online-softmax state;
// the phases are merged with wavefront shuffles at the end.  All accumulation is fp32.
// The head dimension (8, 16, 32, 64) is a template parameter; the LDS tiles hold b rows and are
// sized at launch.  With the full short-term mask of Eq. 15 and a mask block smaller than b, the
// far keys of each row (power-of-two distances, last block) are read straight from memory by the
// row's own lanes instead of being walked tile by tile.
#include "common.h"
#include "gate_reduce.h"
#include "launch.h"
#include "mfma_common.h"

namespace blossom {

namespace {

constexpr float kNegInf = -__builtin_huge_valf();

template <typename T, int D>
__device__ __forceinline__ void load_row(const T *src, float (&r)[D])
{
#pragma unroll
  for (int c = 0; c < D; c += 4) {
    float x[4];
    load4(src + c, x);
    r[c] = x[0]; r[c + 1] = x[1]; r[c + 2] = x[2]; r[c + 3] = x[3];
  }
}

template <typename T, int D>
__device__ __forceinline__ void store_row(T *dst, const float (&r)[D])
{
#pragma unroll
  for (int c = 0; c < D; c += 4) {
    const float x[4] = {r[c], r[c + 1], r[c + 2], r[c + 3]};
    store4(dst + c, x);
  }
}

// Stage rows [J*b, J*b+b) of one head's [L,D] tensor into LDS as fp32; rows >= L become 0.
template <typename T, int D>
__device__ __forceinline__ void stage_tile(const T *head, int J, int b, int L, float (*dst)[D + 1], int lane)
{
  const int groups = b * (D / 4);
  for (int idx = lane; idx < groups; idx += 64) {
    const int rr = idx / (D / 4);
    const int c4 = (idx % (D / 4)) * 4;
    const int pos = J * b + rr;
    float x[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (pos < L) load4(head + (size_t)pos * D + c4, x);
    dst[rr][c4] = x[0]; dst[rr][c4 + 1] = x[1]; dst[rr][c4 + 2] = x[2]; dst[rr][c4 + 3] = x[3];
  }
}

__device__ __forceinline__ int first_window_block(int I, int b, int w, int J_first)
{
  const int lowpos = I * b - (w - 1);
  const int J = lowpos <= 0 ? 0 : lowpos / b;
  return J > J_first ? J : J_first;
}

// bidirectional form: last key block the window of a query of block I reaches
__device__ __forceinline__ int last_window_block(int I, int b, int w, int NB)
{
  const long hi = (long)I * b + (b - 1) + (w - 1);
  return (int)min((long)(NB - 1), hi / b);
}

// Far part of the short-term mask when the mask block is smaller than the tile (Eq. 15, second and
// third case, below the window tiles): the rows of a query block then see different, short runs of
// keys, so each lane reads its own keys straight from memory instead of walking whole tiles.
// Calls f(j) once for every key j in [p0, far_hi) at a power-of-two mask-block distance from
// query i, or among the last sblk positions; the runs are dealt over the nph phases of the row.
template <typename F>
__device__ __forceinline__ void far_keys_of_row(const KParams &p, int i, int p0, int far_hi, int phase, int nph, F &&f)
{
  const int qb = i / p.sblk;
  for (int r = phase; r < 31; r += nph) {
    const int mb = qb - (1 << r);
    if (mb < 0) break;
    const int lo = max(mb * p.sblk, p0), hi = min(mb * p.sblk + p.sblk, far_hi);
    for (int j = lo; j < hi; ++j) f(j);
  }
  if (phase == 0)
    for (int j = max(p.last_lo, p0); j < far_hi; ++j)
      if (!is_pow2(qb - j / p.sblk)) f(j);
}
// The same pairs from the key's side: f(i) for every query i in [far_lo, L) that sees key j that way.
template <typename F>
__device__ __forceinline__ void far_rows_of_key(const KParams &p, int j, int far_lo, int phase, int nph, F &&f)
{
  const int kb = j / p.sblk;
  for (int r = phase; r < 31; r += nph) {
    const long first = ((long)kb + (1L << r)) * p.sblk;
    if (first >= p.L) break;
    const int lo = max((int)first, far_lo), hi = min((int)first + p.sblk, p.L);
    for (int i = lo; i < hi; ++i) f(i);
  }
  if (phase == 0 && j >= p.last_lo)
    for (int i = far_lo; i < p.L; ++i)
      if (!is_pow2(i / p.sblk - kb)) f(i);
}
// (host side: picks the instantiation)
// (the bidirectional form walks whole tiles on both sides of the query block)
static inline bool far_by_rows(const KParams &p) { return p.sblk > 0 && p.sblk < p.b && !p.bidir; }

}  // namespace

// =============================================================================================
// Forward
// =============================================================================================
// FAR: the far part of the short-term mask is gathered row by row (mask block smaller than the
// tile); a separate instantiation, so that the plain kernels keep their register budget.
template <typename T, int D, bool FAR>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(D <= 32 ? 4 : 2))) void fwd_generic_kernel(const T *__restrict__ Q, const T *__restrict__ K,
                                                         const T *__restrict__ V,
                                                         const int *__restrict__ valid_len,
                                                         const int *__restrict__ sel,
                                                         const float *__restrict__ gate_w,
                                                         const float *__restrict__ gate_b,
                                                         T *__restrict__ O, float *__restrict__ o_lt_out,
                                                         float *__restrict__ o_st_out,
                                                         float *__restrict__ lse_lt_out,
                                                         float *__restrict__ lse_st_out, int dense,
                                                         KParams p)
{
  // three tiles of b rows (sized at launch: with small blocks a fixed 64-row layout would cap the
  // number of resident wavefronts): K, V, and the short-term output of each row, parked during
  // the long-term pass
  extern __shared__ float fwd_lds[];
  const int lane = threadIdx.x;
  const int b = p.b;
  float (*Ks)[D + 1] = reinterpret_cast<float (*)[D + 1]>(fwd_lds);
  float (*Vs)[D + 1] = Ks + b;
  float (*Os)[D + 1] = Vs + b;
  const int nph = 64 / b;
  const int row = lane % b;
  const int phase = lane / b;
  const int bh = blockIdx.x / p.nq;
  const int I = p.NB - 1 - (int)(blockIdx.x % p.nq);  // late (long) blocks first
  const int h = bh % p.H;
  const int n = clamp_len(valid_len[bh / p.H], p.L);
  const int p0 = p.L - n;
  const int i = I * b + row;
  const bool in_range = i < p.L;
  const bool active = in_range && i >= p0;
  const size_t head = (size_t)bh * p.L * D;
  const size_t rowoff = head + (size_t)i * D;
  const size_t lrow = (size_t)bh * p.L + i;

  float acc[D];
  if (min((I + 1) * b, p.L) <= p0) {  // no valid query in the block: outputs are zero
    if (phase == 0 && in_range) {
#pragma unroll
      for (int c = 0; c < D; ++c) acc[c] = 0.0f;
      store_row<T, D>(O + rowoff, acc);
      if (o_lt_out) store_row<float, D>(o_lt_out + rowoff, acc);
      if (o_st_out) store_row<float, D>(o_st_out + rowoff, acc);
      if (lse_lt_out) lse_lt_out[lrow] = 0.0f;
      if (lse_st_out) lse_st_out[lrow] = 0.0f;
    }
    return;
  }

  float q[D];
  if (active) {
    load_row<T, D>(Q + rowoff, q);
  } else {
#pragma unroll
    for (int c = 0; c < D; ++c) q[c] = 0.0f;
  }
  const int J_first = p0 / b;
  const T *Kh = K + head;
  const T *Vh = V + head;
  float m, l;

  auto tile = [&](int J, bool windowed) {
    __syncthreads();
    stage_tile<T, D>(Kh, J, b, p.L, Ks, lane);
    stage_tile<T, D>(Vh, J, b, p.L, Vs, lane);
    __syncthreads();
    for (int jj = phase; jj < b; jj += nph) {
      const int j = J * b + jj;
      const bool vis = active && j < p.L && j >= p0 && (j <= i || p.bidir) && (!windowed || st_visible(p, i, j));
      if (vis) {
        float s4[4] = {0.0f, 0.0f, 0.0f, 0.0f};  // four independent chains
#pragma unroll
        for (int c = 0; c < D; ++c) s4[c & 3] = fmaf(q[c], Ks[jj][c], s4[c & 3]);
        const float s = ((s4[0] + s4[1]) + (s4[2] + s4[3])) * p.scale;
        if (s > m) {
          const float corr = __expf(m - s);
          l *= corr;
#pragma unroll
          for (int c = 0; c < D; ++c) acc[c] *= corr;
          m = s;
        }
        const float pj = __expf(s - m);
        l += pj;
#pragma unroll
        for (int c = 0; c < D; ++c) acc[c] = fmaf(pj, Vs[jj][c], acc[c]);
      }
    }
  };

  auto finish = [&]() -> float {  // merge the phases, normalise; returns lse
    for (int off = b; off < 64; off <<= 1) {
      const float m2 = __shfl_xor(m, off);
      const float l2 = __shfl_xor(l, off);
      const float mn = fmaxf(m, m2);
      const float c1 = (m == kNegInf) ? 0.0f : __expf(m - mn);
      const float c2 = (m2 == kNegInf) ? 0.0f : __expf(m2 - mn);
      l = l * c1 + l2 * c2;
#pragma unroll
      for (int c = 0; c < D; ++c) {
        const float a2 = __shfl_xor(acc[c], off);
        acc[c] = acc[c] * c1 + a2 * c2;
      }
      m = mn;
    }
    float lse = 0.0f;
    if (active) {  // the query itself is always visible, so l > 0
      const float inv = 1.0f / l;
#pragma unroll
      for (int c = 0; c < D; ++c) acc[c] *= inv;
      lse = m + logf(l);
    } else {
#pragma unroll
      for (int c = 0; c < D; ++c) acc[c] = 0.0f;
    }
    return lse;
  };

  auto reset = [&]() {
    m = kNegInf;
    l = 0.0f;
#pragma unroll
    for (int c = 0; c < D; ++c) acc[c] = 0.0f;
  };

  if (dense) {
    reset();
    for (int J = J_first; J <= I; ++J) tile(J, false);
    const float lse = finish();
    if (phase == 0 && in_range) {
      store_row<T, D>(O + rowoff, acc);
      if (lse_lt_out) lse_lt_out[lrow] = lse;
    }
    return;
  }

  // ---- short-term branch: causal window, plus the keys the other cases of Eq. 15 reach ----
  reset();
  {
    const int J_win = first_window_block(I, b, p.w, J_first);
    if constexpr (FAR) {
      if (active)
        far_keys_of_row(p, i, p0, J_win * b, phase, nph, [&](int j) {
          const T *kp = Kh + (size_t)j * D, *vp = Vh + (size_t)j * D;
          float s4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int c = 0; c < D; c += 4) {
            float x[4];
            load4(kp + c, x);
#pragma unroll
            for (int e = 0; e < 4; ++e) s4[e] = fmaf(q[c + e], x[e], s4[e]);
          }
          const float s = ((s4[0] + s4[1]) + (s4[2] + s4[3])) * p.scale;
          if (s > m) {
            const float corr = __expf(m - s);
            l *= corr;
#pragma unroll
            for (int c = 0; c < D; ++c) acc[c] *= corr;
            m = s;
          }
          const float pj = __expf(s - m);
          l += pj;
#pragma unroll
          for (int c = 0; c < D; c += 4) {
            float x[4];
            load4(vp + c, x);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[c + e] = fmaf(pj, x[e], acc[c + e]);
          }
        });
    } else {
      for (int J = J_first; J < J_win; ++J)
        if (st_block_reach(p, I, J)) tile(J, true);
    }
    for (int J = J_win; J <= I; ++J) tile(J, true);
    if (p.bidir) {  // Eq. 15 as printed: the same on the other side of the query block
      const int J_whi = last_window_block(I, b, p.w, p.NB);
      for (int J = I + 1; J < p.NB; ++J)
        if (J <= J_whi || st_block_reach(p, I, J)) tile(J, true);
    }
  }
  const float lse_st = finish();
  float z = gate_b ? gate_b[h] : 0.0f;
  if (phase == 0) {
    const float *ws = gate_w + (size_t)h * 2 * D + D;
#pragma unroll
    for (int c = 0; c < D; ++c) {
      Os[row][c] = acc[c];
      z = fmaf(ws[c], acc[c], z);
    }
    if (in_range) {
      if (o_st_out) store_row<float, D>(o_st_out + rowoff, acc);
      if (lse_st_out) lse_st_out[lrow] = lse_st;
    }
  }

  // ---- long-term branch: selected blocks ----
  reset();
  const int *my_sel = sel + ((size_t)bh * p.NB + I) * p.k;
  for (int e = 0; e < p.k; ++e) {
    const int J = my_sel[e];
    if (J < 0 || J >= p.NB) continue;
    tile(J, false);
  }
  const float lse_lt = finish();

  // ---- gate and blend (Eq. 18-19) ----
  if (phase == 0 && in_range) {
    if (o_lt_out) store_row<float, D>(o_lt_out + rowoff, acc);
    if (lse_lt_out) lse_lt_out[lrow] = lse_lt;
    const float *wl = gate_w + (size_t)h * 2 * D;
#pragma unroll
    for (int c = 0; c < D; ++c) z = fmaf(wl[c], acc[c], z);
    const float alpha = active ? 1.0f / (1.0f + __expf(-z)) : 0.0f;
#pragma unroll
    for (int c = 0; c < D; ++c) acc[c] = alpha * acc[c] + (1.0f - alpha) * Os[row][c];
    store_row<T, D>(O + rowoff, acc);
  }
}

// =============================================================================================
// Backward: inverse selection list.  For each key block J of a (row, head): the list of
// query blocks I whose selection holds J, in a fixed, deterministic order.
// offs [B*H,(NB+1)], items [B*H,NB*k].
// One workgroup of W wavefronts per (row, head); wavefront w owns a contiguous range of query
// blocks and its own counters.  Counting and filling use LDS integer atomics, one selection
// row per wavefront instruction: a row lists distinct blocks, and the LDS executes one
// wavefront's instructions in order, so the order inside a wavefront's range is that of the
// fill loop: by 64-entry chunk of the selection row, then by I (ascending in I whenever
// topk <= 64); the ranges are laid out one after the other per key block (the scan hands each
// wavefront its base).  The consumers sum over the list and need no particular order, only the
// same one on every run.
// =============================================================================================
constexpr int kInvWaves = 4;      // wavefronts per (row, head) when the counters fit
constexpr int kInvWavesMaxNB = 2048;

// lds: cnt[W][NB+1], then few[NB+1] bytes
__device__ __forceinline__ void inverse_list(const int *__restrict__ sel, const int *__restrict__ valid_len, int *__restrict__ offs,
                                             int *__restrict__ items, const KParams &p, int bh, int *inv_lds)
{
  const int W = blockDim.x >> 6;
  const int stride = p.NB + 1;
  int *cnt = inv_lds;
  unsigned char *few = reinterpret_cast<unsigned char *>(inv_lds + W * stride);  // query block whose selected
                                                                                  // past blocks hold few valid keys
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wv = tid >> 6;
  const int *s = sel + (size_t)bh * p.NB * p.k;
  int *o = offs + (size_t)bh * (p.NB + 1);
  int *it = items + (size_t)bh * p.NB * p.k;
  const int p0 = p.L - clamp_len(valid_len[bh / p.H], p.L);
  const int per = (p.NB + W - 1) / W;
  const int I_lo = wv * per, I_hi = min(p.NB, I_lo + per);
  int *mine = cnt + wv * stride;
  // entry e of each of the wavefront's rows in turn, eight rows on their way at a time (one load a row, waited for, before)
  auto each_row = [&](int e, auto f) __attribute__((always_inline)) {
    for (int I0 = I_lo; I0 < I_hi; I0 += 8) {
      int J[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) J[i] = s[(size_t)min(I0 + i, I_hi - 1) * p.k + min(e, p.k - 1)];
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (I0 + i < I_hi) f(I0 + i, e < p.k ? J[i] : -1);
    }
  };
  for (int x = tid; x < W * stride; x += blockDim.x) cnt[x] = 0;
  for (int J = tid; J <= p.NB; J += blockDim.x) few[J] = 1;
  __syncthreads();
  for (int e0 = 0; e0 < p.k; e0 += 64) {
    const int e = e0 + lane;
    each_row(e, [&](int I, int J) __attribute__((always_inline)) {
      if (J >= 0 && J < p.NB && (J <= I || p.bidir)) atomicAdd(&mine[J], 1);
      // an earlier block with at least kInvFewKeys valid keys gives every row of I that many keys
      const int vcount = min((J + 1) * p.b, p.L) - max(J * p.b, p0);
      if (__ballot(J >= 0 && J < I && vcount >= kInvFewKeys) != 0ull && lane == 0) few[I] = 0;
    });
  }
  __syncthreads();
  // exclusive scan over (key block, wavefront) in chunks of 64 key blocks; o[NB] receives the total
  if (wv == 0) {
    int carry = 0;
    for (int J0 = 0; J0 <= p.NB; J0 += 64) {
      const int J = J0 + lane;
      int c = 0;
      if (J < p.NB)
        for (int w = 0; w < W; ++w) c += cnt[w * stride + J];
      int incl = c;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const int up = __shfl_up(incl, off);
        if (lane >= off) incl += up;
      }
      if (J <= p.NB) {
        int base = carry + incl - c;
        o[J] = base;
        if (J < p.NB)
          for (int w = 0; w < W; ++w) {
            const int cw = cnt[w * stride + J];
            cnt[w * stride + J] = base;
            base += cw;
          }
      }
      carry += __shfl(incl, 63);
    }
  }
  __syncthreads();
  for (int e0 = 0; e0 < p.k; e0 += 64) {
    const int e = e0 + lane;
    each_row(e, [&](int I, int J) __attribute__((always_inline)) {
      if (J >= 0 && J < p.NB && (J <= I || p.bidir)) it[atomicAdd(&mine[J], 1)] = I | ((int)few[I] << kInvFewShift);
    });
  }
}
size_t inverse_list_lds(const KParams &p, int W) { return (size_t)W * (p.NB + 1) * sizeof(int) + (size_t)(p.NB + 1 + 3) / 4 * 4; }

__global__ __launch_bounds__(64 * kInvWaves) void inverse_list_kernel(const int *__restrict__ sel,
                                                                      const int *__restrict__ valid_len,
                                                                      int *__restrict__ offs, int *__restrict__ items,
                                                                      KParams p)
{
  extern __shared__ int inv_lds[];
  inverse_list(sel, valid_len, offs, items, p, blockIdx.x, inv_lds);
}

// =============================================================================================
// Backward, step 1: gate backward per row + per-chunk partial gate-weight gradients.
//   rowstat[row] = (alpha, dz, D_lt, D_st); in the matrix-core path (y_lt, y_st, -c_lt, -c_st) and rowI_x the row constants of
//   branch x, see below
//   partial[(bh*nchunk+chunk)][0..2D] (2D = bias)
// Every tensor is read exactly once, so memory is the bound, but a row costs five sums over its channels and
// some sixty instructions that its lanes share: as few lanes as give whole cache lines take a row (4 channels
// each, for d = 64 twice 4: 8 lanes), the sums are DPP adds inside a row of 16 lanes instead of LDS permutes, and the
// next rows are requested before the current ones are worked on.  B=128 H=4 L=1024 d=64, lengths U[100,1024]: 77 -> 71 us, 59 with the
// heads to the XCDs in turn; B=16 H=8 L=8192: 183 -> 175 us (5.7 TB/s).  Since it writes no gradients of the branches for the
// matrix-core kernels, 52 and 148 us; with chunks of 64 rows, whose last ones leave fewer CUs idle than those of 128, and the lists'
// rows eight at a time, 48 and 142; with a chunk's two steps written out 45 and 124 (47 and 131 in the same run; 5.9 TB/s of
// the 738 MB that it moves there).  What a short batch loses is its padding: workgroups that find no valid row, and the last ones of each head.
// The gate-weight partials accumulate in registers and meet in LDS in a fixed order.
// =============================================================================================
// The first `lists` workgroups make the inverse selection lists instead: a chain of latencies (8 us at B=128 H=4 L=1024, 26 at B=16
// H=8 L=8192 as a launch of its own) beside work that waits for memory.
// Rows of a chunk: as many as the workgroup takes in two steps (d >= 32) or in one.
__host__ __device__ constexpr int prep_rows(int d) { return d == 8 ? 128 : 64; }
// Branch outputs from a quarter of the last-level cache on leave it to Q, K, V and dO, which the kernels that follow read: a training
// step at B=32 H=8 L=700 d=64 b=32 113.5 -> 106.5 us, B=128 H=4 L=1024 324 -> 312.5, B=16 H=8 L=8192 1907 -> 1900; at B=16 H=8 L=500
// (33 MB) 57.8 without and 58.4 with.
constexpr size_t kBranchesOnceBytes = 64u << 20;
constexpr size_t kPrepListLds = 8320;  // LDS that every head size has for them: up to 488 blocks

// four consecutive elements as loaded, and as floats (zeros unless `keep`)
struct Raw4f { uint4 w; };
struct Raw4h { uint2 w; };
__device__ __forceinline__ Raw4f load_raw4(const float *p) { return {*reinterpret_cast<const uint4 *>(p)}; }
__device__ __forceinline__ Raw4h load_raw4(const bf16_t *p) { return {*reinterpret_cast<const uint2 *>(p)}; }
__device__ __forceinline__ void unpack4(Raw4f r, bool keep, float *o)
{
  o[0] = __uint_as_float(keep ? r.w.x : 0u); o[1] = __uint_as_float(keep ? r.w.y : 0u);
  o[2] = __uint_as_float(keep ? r.w.z : 0u); o[3] = __uint_as_float(keep ? r.w.w : 0u);
}
__device__ __forceinline__ void unpack4(Raw4h r, bool keep, float *o)
{
  const uint32_t x = keep ? r.w.x : 0u, y = keep ? r.w.y : 0u;
  o[0] = mfma::bf_lo(x); o[1] = mfma::bf_hi(x); o[2] = mfma::bf_lo(y); o[3] = mfma::bf_hi(y);
}

template <int CTRL>
__device__ __forceinline__ float dpp_of(float x)
{
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false));
}
// sum over N = 2, 4, 8 or 16 adjacent lanes, the same in all of them
template <int N>
__device__ __forceinline__ float lanes_sum(float x)
{
  x += dpp_of<0xB1>(x);                  // the neighbour
  if (N > 2) x += dpp_of<0x4E>(x);       // the other pair of the quad
  if (N > 4) x += dpp_of<0x141>(x);      // half-row mirror: the other quad (its lanes agree)
  if (N > 8) x += dpp_of<0x140>(x);      // row mirror: the other half
  return x;
}

// STREAM: the branch outputs, which nothing reads again, are read past the caches (see kBranchesOnceBytes).
template <typename T, int D, bool STREAM>
__global__ __launch_bounds__(256) void bwd_prep_kernel(const float *__restrict__ o_lt,
                                                       const float *__restrict__ o_st,
                                                       const T *__restrict__ dO,
                                                       const int *__restrict__ valid_len,
                                                       const float *__restrict__ gate_w,
                                                       const float *__restrict__ gate_b,
                                                       float4 *__restrict__ rowstat,
                                                       float *__restrict__ partial,
                                                       const float *__restrict__ lse_lt,
                                                       const float *__restrict__ lse_st,
                                                       uint4 *__restrict__ rowI_lt,
                                                       uint4 *__restrict__ rowI_st, const int *__restrict__ sel,
                                                       int *__restrict__ offs, int *__restrict__ items, int lists, KParams p)
{
  constexpr int CPL = D >= 64 ? 8 : 4;  // channels per lane, in groups of four D/2 apart
  constexpr int NG = CPL / 4;
  constexpr int LPR = D / CPL;          // lanes per row
  constexpr int RPW = 64 / LPR;         // rows per wavefront step
  constexpr int RPS = 4 * RPW;          // rows per workgroup step
  constexpr int G = 2 * D + 1;
  static_assert(sizeof(float) * 4 * RPW * G >= kPrepListLds && 4 == kInvWaves, "the lists use the same LDS and wavefronts");
  __shared__ float red[4 * RPW][G];
  if ((int)blockIdx.x < lists) {
    inverse_list(sel, valid_len, offs, items, p, blockIdx.x, reinterpret_cast<int *>(&red[0][0]));
    return;
  }
  const int t = threadIdx.x;
  const int wave = t >> 6, lane = t & 63;
  const int sub = lane % LPR, rg = lane / LPR;
  const int c4 = sub * 4;
  constexpr int ROWS = prep_rows(D);
  static_assert(ROWS % RPS == 0, "whole steps: a row must not be counted in two chunks");
  const int nchunk = (p.L + ROWS - 1) / ROWS;
  // (chunk by chunk the workgroups would go to the XCDs in turn, and where there are eight chunks to a head, or a multiple, one XCD
  // would have the last, always valid ones to do and another nothing but padding)
  const unsigned vid = mfma::xcd_spread(blockIdx.x - lists, (gridDim.x - lists) / nchunk, nchunk);
  const int bh = (int)(vid / nchunk);
  const int chunk = (int)(vid % nchunk);
  const int h = bh % p.H;
  const int n = clamp_len(valid_len[bh / p.H], p.L);
  const int p0 = p.L - n;
  // rows of blocks that hold no valid position are never read by the kernels that follow: nothing is
  // written for them (pad rows of a partly valid block are staged with their tile and get zeros)
  const int first = (p0 / p.b) * p.b;
  float *out = partial + (size_t)vid * G;
  if ((chunk + 1) * ROWS <= first) {
    for (int c = t; c < G; c += 256) out[c] = 0.0f;
    return;
  }
  const size_t head = (size_t)bh * p.L * D;

  struct Rows {
    decltype(load_raw4(dO)) g[NG];
    Raw4f ol[NG], os[NG];
    float ll, ls;
  };
  const int row0 = chunk * ROWS + wave * RPW + rg;
  auto request = [&](int base, Rows &r) __attribute__((always_inline)) {
    const int i = min(max(row0 + base, p0), p.L - 1);
    const size_t ro = head + (size_t)i * D + c4, lr = (size_t)bh * p.L + i;
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      r.g[q] = load_raw4(dO + ro + q * (D / 2));
      if constexpr (STREAM) {
        r.ol[q] = {load_once(reinterpret_cast<const uint4 *>(o_lt + ro + q * (D / 2)))};
        r.os[q] = {load_once(reinterpret_cast<const uint4 *>(o_st + ro + q * (D / 2)))};
      } else {
        r.ol[q] = load_raw4(o_lt + ro + q * (D / 2));
        r.os[q] = load_raw4(o_st + ro + q * (D / 2));
      }
    }
    r.ll = r.ls = 0.0f;
    if (rowI_lt) {
      r.ll = lse_lt[lr];
      r.ls = lse_st[lr];
    }
  };
  Rows cur, nxt;
  request(0, cur);
  float wl[CPL], ws[CPL];
#pragma unroll
  for (int q = 0; q < NG; ++q) {
    unpack4(load_raw4(gate_w + (size_t)h * 2 * D + c4 + q * (D / 2)), true, wl + 4 * q);
    unpack4(load_raw4(gate_w + (size_t)h * 2 * D + D + c4 + q * (D / 2)), true, ws + 4 * q);
  }
  const float bias = gate_b ? gate_b[h] : 0.0f;
  float acc_l[CPL], acc_s[CPL], acc_b = 0.0f;
#pragma unroll
  for (int e = 0; e < CPL; ++e) acc_l[e] = acc_s[e] = 0.0f;

  // (both steps written out, at d = 32 and 64; below, a chunk is one step: 86 instead of 105 registers at d = 64 in bf16, 90 instead of 109 in
  // fp32, where the copies of a loop keep two sets of rows alive to its end: five wavefronts a SIMD instead of four)
#pragma unroll
  for (int base = 0; base < ROWS; base += RPS) {
    const int i = row0 + base;
    const bool valid = i < p.L && i >= p0;
    const bool inb = i < p.L && i >= first;
    if (base + RPS < ROWS) request(base + RPS, nxt);
    float g[CPL], ol[CPL], os[CPL];
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      unpack4(cur.g[q], valid, g + 4 * q);
      unpack4(cur.ol[q], valid, ol + 4 * q);
      unpack4(cur.os[q], valid, os + 4 * q);
    }
    const float ll = cur.ll, ls = cur.ls;
    cur = nxt;
    float a_ll = 0.f, a_ss = 0.f, w_l = 0.f, w_s = 0.f;
#pragma unroll
    for (int e = 0; e < CPL; ++e) {
      a_ll = fmaf(g[e], ol[e], a_ll);
      a_ss = fmaf(g[e], os[e], a_ss);
      w_l = fmaf(wl[e], ol[e], w_l);
      w_s = fmaf(ws[e], os[e], w_s);
    }
    a_ll = lanes_sum<LPR>(a_ll);
    a_ss = lanes_sum<LPR>(a_ss);
    w_l = lanes_sum<LPR>(w_l);
    w_s = lanes_sum<LPR>(w_s);
    float4 st = make_float4(0.f, 0.f, 0.f, 0.f);
    float dz = 0.0f, alpha = 0.0f;
    if (valid) {
      const float z = bias + w_l + w_s;
      alpha = 1.0f / (1.0f + __expf(-z));
      dz = (a_ll - a_ss) * alpha * (1.0f - alpha);
      st = make_float4(alpha, dz, alpha * a_ll + dz * w_l, (1.0f - alpha) * a_ss + dz * w_s);
    }
    if (rowI_lt) {
      // Matrix-core path: the upstream gradient of branch x is a_x*(dO + y_x*Wg_x), a_lt = alpha, a_st = 1 - alpha, y_lt = (1-alpha)*t,
      // y_st = alpha*t, t = dO.(o_lt - o_st); y_x as the two bf16 terms that the kernels read.  Two row constants stand beside it:
      // D_x = (dO + y_x*Wg_x).o_x, and c_x, the same with the bracket rounded to bf16, as dQ takes it.  rowI_x (x: s0 s1, y: D2 s2,
      // z: D0 D1, w: y0 y1): the three-term bf16 splits of -lse*log2(e) + log2(a_x) and of -D_x and the terms of y_x, in the
      // order in which one matrix instruction takes them.
      const float t = a_ll - a_ss;
      const uint32_t yl2 = mfma::split2((1.0f - alpha) * t), ys2 = mfma::split2(alpha * t);
      const float yl = mfma::unsplit2(yl2), ys = mfma::unsplit2(ys2);
      float c_l = 0.0f, c_s = 0.0f;
#pragma unroll
      for (int e = 0; e < CPL; e += 2) {
        const uint32_t gl = mfma::pack2_bf16(fmaf(yl, wl[e], g[e]), fmaf(yl, wl[e + 1], g[e + 1]));
        const uint32_t gs = mfma::pack2_bf16(fmaf(ys, ws[e], g[e]), fmaf(ys, ws[e + 1], g[e + 1]));
        c_l = fmaf(mfma::bf_hi(gl), ol[e + 1], fmaf(mfma::bf_lo(gl), ol[e], c_l));
        c_s = fmaf(mfma::bf_hi(gs), os[e + 1], fmaf(mfma::bf_lo(gs), os[e], c_s));
      }
      c_l = lanes_sum<LPR>(c_l);
      c_s = lanes_sum<LPR>(c_s);
      st = make_float4(valid ? yl : 0.0f, valid ? ys : 0.0f, valid ? -c_l : 0.0f, valid ? -c_s : 0.0f);
      if (inb && sub < 2) {  // lane 0 of the row writes the long-term constants, lane 1 the short-term ones
        const size_t r = (size_t)bh * p.L + i;
        const float a = sub == 0 ? alpha : 1.0f - alpha;
        // an exponent of -1e30 makes every probability of the row zero: of pad rows, and of a branch whose weight is (log2 of it:
        // the probabilities come out multiplied by the weight)
        const float e2 = -(sub == 0 ? ll : ls) * 1.4426950408889634f + __log2f(a);
        const uint2 l = mfma::split3(valid && !(a < 1.17549435e-38f) ? e2 : -1.0e30f);
        const uint2 k = mfma::split3(valid ? -(sub == 0 ? fmaf(yl, w_l, a_ll) : fmaf(ys, w_s, a_ss)) : 0.0f);
        (sub == 0 ? rowI_lt : rowI_st)[r] = make_uint4(l.x, k.y | l.y << 16, k.x, valid ? (sub == 0 ? yl2 : ys2) : 0u);
      }
    }
    if (inb && sub == 0) rowstat[(size_t)bh * p.L + i] = st;
#pragma unroll
    for (int e = 0; e < CPL; ++e) {
      acc_l[e] = fmaf(dz, ol[e], acc_l[e]);
      acc_s[e] = fmaf(dz, os[e], acc_s[e]);
    }
    acc_b += dz;
  }
  const int slot = wave * RPW + rg;
#pragma unroll
  for (int e = 0; e < CPL; ++e) {
    const int c = c4 + (e & 3) + (e >> 2) * (D / 2);
    red[slot][c] = acc_l[e];
    red[slot][D + c] = acc_s[e];
  }
  if (sub == 0) red[slot][2 * D] = acc_b;
  __syncthreads();
  for (int c = t; c < G; c += 256) {
    float acc = 0.0f;
#pragma unroll
    for (int sl = 0; sl < 4 * RPW; ++sl) acc += red[sl][c];
    out[c] = acc;
  }
}

// The partial gate gradients' sum, where no other kernel takes it along.  One launch: at these sizes (a few MB at most) a second
// level costs more in launching (4-5 us) than it saves in reading.
constexpr int kGateCols = 16;

__global__ __launch_bounds__(1024) void bwd_gate_reduce_kernel(const float *__restrict__ partial,
                                                               float *__restrict__ d_gate_w,
                                                               float *__restrict__ d_gate_b, int nchunk, KParams p)
{
  __shared__ float red[kGateRows][kGateCols + 1];
  gate_reduce<1024, kGateCols>(partial, d_gate_w, d_gate_b, nchunk, p, blockIdx.x, blockIdx.y * kGateCols, red);
}

// =============================================================================================
// Backward, step 2: dQ (query-block stationary, same tile walk as the forward).
//   dP_ij = dO_x[i].v_j = a_x[i]*(dO[i].v_j) + dz[i]*(gate_w_x.v_j)
// =============================================================================================
template <typename T, int D, bool FAR>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(D <= 32 ? 3 : 1))) void bwd_dq_generic_kernel(const T *__restrict__ Q, const T *__restrict__ K,
                                                            const T *__restrict__ V,
                                                            const int *__restrict__ valid_len,
                                                            const int *__restrict__ sel,
                                                            const float *__restrict__ gate_w,
                                                            const float *__restrict__ lse_lt,
                                                            const float *__restrict__ lse_st,
                                                            const T *__restrict__ dO,
                                                            const float4 *__restrict__ rowstat,
                                                            T *__restrict__ dQ, KParams p)
{
  extern __shared__ float dq_lds[];  // K and V tiles of b rows (sized at launch)
  __shared__ float wv[64];           // gate_w_x . v_j of the staged tile

  const int lane = threadIdx.x;
  const int b = p.b;
  float (*Ks)[D + 1] = reinterpret_cast<float (*)[D + 1]>(dq_lds);
  float (*Vs)[D + 1] = Ks + b;
  const int nph = 64 / b;
  const int row = lane % b;
  const int phase = lane / b;
  const int bh = blockIdx.x / p.NB;
  const int I = p.NB - 1 - (int)(blockIdx.x % p.NB);
  const int h = bh % p.H;
  const int n = clamp_len(valid_len[bh / p.H], p.L);
  const int p0 = p.L - n;
  const int i = I * b + row;
  const bool in_range = i < p.L;
  const bool active = in_range && i >= p0;
  const size_t head = (size_t)bh * p.L * D;
  const size_t rowoff = head + (size_t)i * D;

  float dq[D];
#pragma unroll
  for (int c = 0; c < D; ++c) dq[c] = 0.0f;
  if (min((I + 1) * b, p.L) <= p0) {
    if (phase == 0 && in_range) store_row<T, D>(dQ + rowoff, dq);
    return;
  }
  float q[D], g[D];
  float4 st = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  float l_lt = 0.0f, l_st = 0.0f;
  if (active) {
    load_row<T, D>(Q + rowoff, q);
    load_row<T, D>(dO + rowoff, g);
    st = rowstat[(size_t)bh * p.L + i];
    l_lt = lse_lt[(size_t)bh * p.L + i];
    l_st = lse_st[(size_t)bh * p.L + i];
  } else {
#pragma unroll
    for (int c = 0; c < D; ++c) { q[c] = 0.0f; g[c] = 0.0f; }
  }
  const int J_first = p0 / b;
  const T *Kh = K + head;
  const T *Vh = V + head;

  auto tile = [&](int J, bool windowed) {
    const float *wx = gate_w + (size_t)h * 2 * D + (windowed ? D : 0);
    const float a_x = windowed ? 1.0f - st.x : st.x;
    const float D_x = windowed ? st.w : st.z;
    const float lse = windowed ? l_st : l_lt;
    __syncthreads();
    stage_tile<T, D>(Kh, J, b, p.L, Ks, lane);
    stage_tile<T, D>(Vh, J, b, p.L, Vs, lane);
    __syncthreads();
    if (lane < b) {
      float a = 0.0f;
      for (int c = 0; c < D; ++c) a = fmaf(wx[c], Vs[lane][c], a);
      wv[lane] = a;
    }
    __syncthreads();
    for (int jj = phase; jj < b; jj += nph) {
      const int j = J * b + jj;
      const bool vis = active && j < p.L && j >= p0 && (j <= i || p.bidir) && (!windowed || st_visible(p, i, j));
      if (vis) {
        float s = 0.0f, gv = 0.0f;
#pragma unroll
        for (int c = 0; c < D; ++c) {
          s = fmaf(q[c], Ks[jj][c], s);
          gv = fmaf(g[c], Vs[jj][c], gv);
        }
        const float pj = __expf(s * p.scale - lse);
        const float dS = pj * (a_x * gv + st.y * wv[jj] - D_x);
#pragma unroll
        for (int c = 0; c < D; ++c) dq[c] = fmaf(dS, Ks[jj][c], dq[c]);
      }
    }
  };

  {
    const int J_win = first_window_block(I, b, p.w, J_first);
    if constexpr (FAR) {
      const float *wx = gate_w + (size_t)h * 2 * D + D;
      if (active)
        far_keys_of_row(p, i, p0, J_win * b, phase, nph, [&](int j) {
          const T *kp = Kh + (size_t)j * D, *vp = Vh + (size_t)j * D;
          float s4[4] = {0.0f, 0.0f, 0.0f, 0.0f}, g4[4] = {0.0f, 0.0f, 0.0f, 0.0f}, w4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int c = 0; c < D; c += 4) {
            float kx[4], vx[4];
            load4(kp + c, kx);
            load4(vp + c, vx);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              s4[e] = fmaf(q[c + e], kx[e], s4[e]);
              g4[e] = fmaf(g[c + e], vx[e], g4[e]);
              w4[e] = fmaf(wx[c + e], vx[e], w4[e]);
            }
          }
          const float sj = (s4[0] + s4[1]) + (s4[2] + s4[3]);
          const float gv = (g4[0] + g4[1]) + (g4[2] + g4[3]);
          const float wvj = (w4[0] + w4[1]) + (w4[2] + w4[3]);
          const float pj = __expf(sj * p.scale - l_st);
          const float dS = pj * ((1.0f - st.x) * gv + st.y * wvj - st.w);
#pragma unroll
          for (int c = 0; c < D; c += 4) {
            float kx[4];
            load4(kp + c, kx);
#pragma unroll
            for (int e = 0; e < 4; ++e) dq[c + e] = fmaf(dS, kx[e], dq[c + e]);
          }
        });
    } else {
      for (int J = J_first; J < J_win; ++J)
        if (st_block_reach(p, I, J)) tile(J, true);
    }
    for (int J = J_win; J <= I; ++J) tile(J, true);
    if (p.bidir) {  // Eq. 15 as printed: the same on the other side of the query block
      const int J_whi = last_window_block(I, b, p.w, p.NB);
      for (int J = I + 1; J < p.NB; ++J)
        if (J <= J_whi || st_block_reach(p, I, J)) tile(J, true);
    }
  }
  const int *my_sel = sel + ((size_t)bh * p.NB + I) * p.k;
  for (int e = 0; e < p.k; ++e) {
    const int J = my_sel[e];
    if (J < 0 || J >= p.NB) continue;
    tile(J, false);
  }
  for (int off = b; off < 64; off <<= 1) {
#pragma unroll
    for (int c = 0; c < D; ++c) dq[c] += __shfl_xor(dq[c], off);
  }
  if (phase == 0 && in_range) {
#pragma unroll
    for (int c = 0; c < D; ++c) dq[c] *= p.scale;
    unrope_row<D>(p, i, dq);
    store_row<T, D>(dQ + rowoff, dq);
  }
}

// =============================================================================================
// Backward, step 4: dK / dV (key-block stationary).  MODE 0 computes dV, 1 dK, 2 both.  With
// d >= 32 they are one launch each: the dV pass needs neither the V row nor the dP product, so it
// runs with fewer registers and more wavefronts; with small d one pass holds both.
// A lane owns one key row and one phase of the query tile.
// =============================================================================================
template <typename T, int D, int MODE, bool FAR>
__global__ __launch_bounds__(64) void bwd_dkv_generic_kernel(const T *__restrict__ Q, const T *__restrict__ K,
                                                             const T *__restrict__ V,
                                                             const int *__restrict__ valid_len,
                                                             const float *__restrict__ gate_w,
                                                             const float *__restrict__ lse_lt,
                                                             const float *__restrict__ lse_st,
                                                             const T *__restrict__ dO,
                                                             const float4 *__restrict__ rowstat,
                                                             const int *__restrict__ offs,
                                                             const int *__restrict__ items,
                                                             T *__restrict__ dK, T *__restrict__ dV,
                                                             KParams p)
{
  extern __shared__ float dkv_lds[];  // Q and dO_x tiles of b rows (sized at launch)
  __shared__ float lse_s[64];
  __shared__ float Dx_s[64];

  const int lane = threadIdx.x;
  const int b = p.b;
  float (*Qs)[D + 1] = reinterpret_cast<float (*)[D + 1]>(dkv_lds);
  float (*Gs)[D + 1] = Qs + b;  // dO_x rows of the staged query tile
  const int nph = 64 / b;
  const int jj = lane % b;
  const int phase = lane / b;
  const int bh = blockIdx.x / p.NB;
  const int J = (int)(blockIdx.x % p.NB);
  constexpr bool want_dk = MODE != 0, want_dv = MODE != 1;
  const int h = bh % p.H;
  const int n = clamp_len(valid_len[bh / p.H], p.L);
  const int p0 = p.L - n;
  const int j = J * b + jj;
  const bool in_range = j < p.L;
  const bool key_ok = in_range && j >= p0;
  const size_t head = (size_t)bh * p.L * D;
  const size_t outoff = head + (size_t)j * D;

  float acck[D], accv[D];
#pragma unroll
  for (int c = 0; c < D; ++c) { acck[c] = 0.0f; accv[c] = 0.0f; }
  if (min((J + 1) * b, p.L) <= p0) {  // no valid key in the block
    if (phase == 0 && in_range) {
      if (want_dk) store_row<T, D>(dK + outoff, acck);
      if (want_dv) store_row<T, D>(dV + outoff, accv);
    }
    return;
  }
  float kr[D], vr[D];
  if (key_ok) {
    load_row<T, D>(K + head + (size_t)j * D, kr);
    if (want_dk) load_row<T, D>(V + head + (size_t)j * D, vr);
  } else {
#pragma unroll
    for (int c = 0; c < D; ++c) { kr[c] = 0.0f; vr[c] = 0.0f; }
  }
  const T *Qh = Q + head;
  const T *Gh = dO + head;

  auto tile = [&](int I, bool windowed) {
    const float *wx = gate_w + (size_t)h * 2 * D + (windowed ? D : 0);
    __syncthreads();
    stage_tile<T, D>(Qh, I, b, p.L, Qs, lane);
    // dO_x = a_x*dO + dz*gate_w_x, formed while staging
    const int groups = b * (D / 4);
    for (int idx = lane; idx < groups; idx += 64) {
      const int rr = idx / (D / 4);
      const int c4 = (idx % (D / 4)) * 4;
      const int pos = I * b + rr;
      float x[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      if (pos < p.L && pos >= p0) {
        load4(Gh + (size_t)pos * D + c4, x);
        const float4 st = rowstat[(size_t)bh * p.L + pos];
        const float a_x = windowed ? 1.0f - st.x : st.x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = a_x * x[e] + st.y * wx[c4 + e];
      }
      Gs[rr][c4] = x[0]; Gs[rr][c4 + 1] = x[1]; Gs[rr][c4 + 2] = x[2]; Gs[rr][c4 + 3] = x[3];
    }
    if (lane < b) {
      const int pos = I * b + lane;
      float l = 0.0f, dx = 0.0f;
      if (pos < p.L && pos >= p0) {
        const float4 st = rowstat[(size_t)bh * p.L + pos];
        l = windowed ? lse_st[(size_t)bh * p.L + pos] : lse_lt[(size_t)bh * p.L + pos];
        dx = windowed ? st.w : st.z;
      }
      lse_s[lane] = l;
      Dx_s[lane] = dx;
    }
    __syncthreads();
    for (int ii = phase; ii < b; ii += nph) {
      const int i = I * b + ii;
      const bool vis = key_ok && i < p.L && i >= p0 && (j <= i || p.bidir) && (!windowed || st_visible(p, i, j));
      if (vis) {
        float s4[4] = {0.0f, 0.0f, 0.0f, 0.0f};  // four independent chains
#pragma unroll
        for (int c = 0; c < D; ++c) s4[c & 3] = fmaf(Qs[ii][c], kr[c], s4[c & 3]);
        const float s = (s4[0] + s4[1]) + (s4[2] + s4[3]);
        const float pj = __expf(s * p.scale - lse_s[ii]);
        if (want_dk) {
          float d4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int c = 0; c < D; ++c) d4[c & 3] = fmaf(Gs[ii][c], vr[c], d4[c & 3]);
          const float dP = (d4[0] + d4[1]) + (d4[2] + d4[3]);
          const float dS = pj * (dP - Dx_s[ii]);
#pragma unroll
          for (int c = 0; c < D; ++c) acck[c] = fmaf(dS, Qs[ii][c], acck[c]);
        }
        if (want_dv) {
#pragma unroll
          for (int c = 0; c < D; ++c) accv[c] = fmaf(pj, Gs[ii][c], accv[c]);
        }
      }
    }
  };

  // short-term branch: query blocks whose window reaches this key block, then those that
  // reach it through the other cases of Eq. 15
  {
    const long last_q = (long)J * b + (b - 1) + (p.w - 1);
    const int I_hi = (int)min((long)(p.NB - 1), last_q / b);
    for (int I = J; I <= I_hi; ++I) tile(I, true);
    if (p.bidir) {  // query blocks before the key block: window reach, then the other cases of Eq. 15
      const int I_first = p0 / b;
      const int I_lo = first_window_block(J, b, p.w, I_first);
      for (int I = I_first; I < J; ++I)
        if (I >= I_lo || st_block_reach(p, I, J)) tile(I, true);
    }
    if constexpr (FAR) {
      const float *wx = gate_w + (size_t)h * 2 * D + D;
      if (key_ok)
        far_rows_of_key(p, j, (I_hi + 1) * b, phase, nph, [&](int i) {
          const size_t r = (size_t)bh * p.L + i;
          const float4 st = rowstat[r];
          const float a_x = 1.0f - st.x;
          const T *qp = Qh + (size_t)i * D, *gp = Gh + (size_t)i * D;
          float s4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int c = 0; c < D; c += 4) {
            float qx[4];
            load4(qp + c, qx);
#pragma unroll
            for (int e = 0; e < 4; ++e) s4[e] = fmaf(qx[e], kr[c + e], s4[e]);
          }
          const float pj = __expf(((s4[0] + s4[1]) + (s4[2] + s4[3])) * p.scale - lse_st[r]);
          float d4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int c = 0; c < D; c += 4) {
            float gx[4];
            load4(gp + c, gx);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float gxe = a_x * gx[e] + st.y * wx[c + e];  // dO_st
              if (want_dk) d4[e] = fmaf(gxe, vr[c + e], d4[e]);
              if (want_dv) accv[c + e] = fmaf(pj, gxe, accv[c + e]);
            }
          }
          if (want_dk) {
            const float dS = pj * (((d4[0] + d4[1]) + (d4[2] + d4[3])) - st.w);
#pragma unroll
            for (int c = 0; c < D; c += 4) {
              float qx[4];
              load4(qp + c, qx);
#pragma unroll
              for (int e = 0; e < 4; ++e) acck[c + e] = fmaf(dS, qx[e], acck[c + e]);
            }
          }
        });
    } else {
      for (int I = I_hi + 1; I < p.NB; ++I)
        if (st_block_reach(p, I, J)) tile(I, true);
    }
  }
  // long-term branch: query blocks that selected this key block
  {
    const int *o = offs + (size_t)bh * (p.NB + 1);
    const int *it = items + (size_t)bh * p.NB * p.k;
    const int e_lo = o[J], e_hi = o[J + 1];
    for (int e = e_lo; e < e_hi; ++e) tile(it[e] & kInvBlockMask, false);
  }
  for (int off = b; off < 64; off <<= 1) {
#pragma unroll
    for (int c = 0; c < D; ++c) {
      if (want_dk) acck[c] += __shfl_xor(acck[c], off);
      if (want_dv) accv[c] += __shfl_xor(accv[c], off);
    }
  }
  if (phase == 0 && in_range) {
    if (want_dk) {
#pragma unroll
      for (int c = 0; c < D; ++c) acck[c] *= p.scale;
      unrope_row<D>(p, j, acck);
      store_row<T, D>(dK + outoff, acck);
    }
    if (want_dv) store_row<T, D>(dV + outoff, accv);
  }
}

// =============================================================================================
// Launchers
// =============================================================================================
template <typename T, int D>
static void launch_fwd_t(const KParams &p, const FwdArgs &a, hipStream_t st)
{
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)(p.B * p.H * p.nq)), dim3(64),
                       3 * (size_t)p.b * (D + 1) * sizeof(float), st,
                       (const T *)a.Q, (const T *)a.K, (const T *)a.V, a.valid_len, a.sel, a.gate_w,
                       a.gate_b, (T *)a.O, (float *)a.o_lt, (float *)a.o_st, a.lse_lt, a.lse_st, a.dense, p);
  };
  if (far_by_rows(p) && !a.dense) go(fwd_generic_kernel<T, D, true>);
  else go(fwd_generic_kernel<T, D, false>);
}

void launch_fwd_generic(const KParams &p, int dtype, const FwdArgs &a, hipStream_t st)
{
  with_head_dim(p.d, [&](auto dim) {
    constexpr int D = decltype(dim)::value;
    if (dtype == 0) launch_fwd_t<float, D>(p, a, st);
    else launch_fwd_t<bf16_t, D>(p, a, st);
  });
}

namespace {
inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
}  // namespace

BwdWorkspace bwd_carve(const KParams &p, int dtype, void *ws)
{
  BwdWorkspace w{};
  char *base = reinterpret_cast<char *>(ws);
  const size_t BH = (size_t)p.B * p.H;
  w.nchunk = (p.L + prep_rows(p.d) - 1) / prep_rows(p.d);
  size_t off = 0;
  w.rowstat = reinterpret_cast<float4 *>(base + off);
  off = align256(off + BH * p.L * sizeof(float4));
  w.offs = reinterpret_cast<int *>(base + off);
  off = align256(off + BH * (p.NB + 1) * sizeof(int));
  w.items = reinterpret_cast<int *>(base + off);
  off = align256(off + BH * p.NB * p.k * sizeof(int));
  w.partial = reinterpret_cast<float *>(base + off);
  off = align256(off + BH * w.nchunk * (2 * p.d + 1) * sizeof(float));
  if (bwd_mfma_supported(p, dtype)) {
    w.rowI_lt = reinterpret_cast<uint4 *>(base + off);
    off = align256(off + BH * p.L * sizeof(uint4));
    w.rowI_st = reinterpret_cast<uint4 *>(base + off);
    off = align256(off + BH * p.L * sizeof(uint4));
  }
  w.total = off;
  return w;
}

size_t bwd_workspace_bytes(const KParams &p, int dtype)
{
  SmallWs w;
  return small_supported(p) ? small_ws_bytes(p, &w, nullptr) : bwd_carve(p, dtype, nullptr).total;
}

static void launch_gate_reduce(const KParams &p, const BwdArgs &a, const float *partial, int nchunk, hipStream_t st)
{
  hipLaunchKernelGGL(bwd_gate_reduce_kernel, dim3((unsigned)p.H, (unsigned)((2 * p.d + kGateCols) / kGateCols)), dim3(1024), 0,
                     st, partial, a.d_gate_w, a.d_gate_b, nchunk, p);
}

static void launch_bwd_small_all(const KParams &p, int dtype, const BwdArgs &a, unsigned stages, int kv_groups, hipStream_t st)
{
  SmallWs w;
  small_ws_bytes(p, &w, reinterpret_cast<char *>(a.ws));
  launch_bwd_small(p, dtype, a, w, stages, kv_groups, st);
  if (launch_failed()) return;
  if (stages & kBwdStageGate) launch_gate_reduce(p, a, w.partial, small_partial_rows(p, dtype, kv_groups), st);
}

void launch_bwd_positions(const KParams &p, int dtype, const BwdArgs &a, int kv_groups, hipStream_t st)
{
  launch_bwd_small_all(p, dtype, a, kBwdStageAll, kv_groups, st);
}

template <typename T, int D>
static void launch_bwd_t(const KParams &p, int dtype, const BwdArgs &a, unsigned stages, hipStream_t st)
{
  const BwdWorkspace w = bwd_carve(p, dtype, a.ws);
  const unsigned BH = (unsigned)(p.B * p.H);
  const bool mfma = bwd_mfma_supported(p, dtype);

  const bool with_lists = (stages & kBwdStageGate) && (stages & kBwdStageInverse) && inverse_list_lds(p, kInvWaves) <= kPrepListLds &&
                          (unsigned long long)BH * (w.nchunk + 1) <= 0x7FFFFFFFull;
  if (stages & kBwdStageGate) {
    const unsigned lists = with_lists ? BH : 0u;
    auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(BH * w.nchunk + lists), dim3(256), 0, st, (const float *)a.o_lt, (const float *)a.o_st,
                         (const T *)a.dO, a.valid_len, a.gate_w, a.gate_b, w.rowstat, w.partial, a.lse_lt, a.lse_st, w.rowI_lt, w.rowI_st,
                         a.sel, w.offs, w.items, (int)lists, p);
    };
    if ((size_t)BH * p.L * 2 * D * sizeof(float) >= kBranchesOnceBytes) go(bwd_prep_kernel<T, D, true>);
    else go(bwd_prep_kernel<T, D, false>);
    if (launch_failed()) return;
    if (!mfma || !bwd_mfma_takes_gate(p, stages)) launch_gate_reduce(p, a, w.partial, w.nchunk, st);
    if (launch_failed()) return;
  }
  if ((stages & kBwdStageInverse) && !with_lists) {
    const int W = p.NB <= kInvWavesMaxNB ? kInvWaves : 1;
    BLOSSOM_LAUNCH(inverse_list_kernel, dim3(BH), dim3(64 * W), inverse_list_lds(p, W), st, a.sel, a.valid_len, w.offs, w.items,
                       p);
  }
  if (mfma) {
    if (launch_failed()) return;
    launch_bwd_mfma(p, a, w, stages, st);
    return;
  }
  const size_t lds = 2 * (size_t)p.b * (D + 1) * sizeof(float);  // two tiles of b rows
  const bool far = far_by_rows(p);
  if (stages & kBwdStageDQ) {
    auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(BH * p.NB), dim3(64), lds, st, (const T *)a.Q, (const T *)a.K,
                         (const T *)a.V, a.valid_len, a.sel, a.gate_w, a.lse_lt, a.lse_st, (const T *)a.dO,
                         w.rowstat, (T *)a.dQ, p);
    };
    if (far) go(bwd_dq_generic_kernel<T, D, true>);
    else go(bwd_dq_generic_kernel<T, D, false>);
    if (launch_failed()) return;
  }
  if (stages & kBwdStageDKV) {
    auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(BH * p.NB), dim3(64), lds, st, (const T *)a.Q, (const T *)a.K,
                         (const T *)a.V, a.valid_len, a.gate_w, a.lse_lt, a.lse_st, (const T *)a.dO, w.rowstat,
                         w.offs, w.items, (T *)a.dK, (T *)a.dV, p);
    };
    if constexpr (D <= 16) {
      if (far) go(bwd_dkv_generic_kernel<T, D, 2, true>);
      else go(bwd_dkv_generic_kernel<T, D, 2, false>);
    } else {
      if (far) {
        go(bwd_dkv_generic_kernel<T, D, 0, true>);
        if (launch_failed()) return;
        go(bwd_dkv_generic_kernel<T, D, 1, true>);
      } else {
        go(bwd_dkv_generic_kernel<T, D, 0, false>);
        if (launch_failed()) return;
        go(bwd_dkv_generic_kernel<T, D, 1, false>);
      }
    }
  }
}

void launch_bwd(const KParams &p, int dtype, const BwdArgs &a, unsigned stages, hipStream_t st)
{
  if (small_supported(p)) {
    launch_bwd_small_all(p, dtype, a, stages, 0, st);
    return;
  }
  with_head_dim(p.d, [&](auto dim) {
    constexpr int D = decltype(dim)::value;
    if (dtype == 0) launch_bwd_t<float, D>(p, dtype, a, stages, st);
    else launch_bwd_t<bf16_t, D>(p, dtype, a, stages, st);
  });
}

}  // namespace blossom
