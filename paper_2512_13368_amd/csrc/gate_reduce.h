// Reduction of the partial gate gradients over batch rows and chunks, by a workgroup of its own kernel or by some workgroups of the
// matrix-core backward, which needs the pass that wrote them but not their sum.
#ifndef BLOSSOM_GATE_REDUCE_H
#define BLOSSOM_GATE_REDUCE_H

#include "common.h"

namespace blossom {

// A workgroup of TH threads closes COLS of the 2d+1 columns of one head, in an order that depends on neither: partial rows n,
// n + 64, ... in four running sums, a tree over the 64 sums of a column.  The rows are few and far apart (B=2048: 2048 of 132 bytes for
// a head of d = 16), so latency is the bound: a thread has sixteen requests on their way, and the row of the next one follows by
// addition.
constexpr int kGateRows = 64;

template <int TH, int COLS>
__device__ __forceinline__ void gate_reduce(const float *__restrict__ partial, float *__restrict__ d_gate_w,
                                            float *__restrict__ d_gate_b, int nchunk, const KParams &p, int h, int c0,
                                            float (*red)[COLS + 1])
{
  constexpr int R = TH / COLS, U = 16;
  static_assert(kGateRows % R == 0 && TH % COLS == 0, "a thread takes whole rows of sums");
  const int G = 2 * p.d + 1;
  const int N = p.B * nchunk;  // partial rows of this head, ordered by (batch row, chunk)
  const int x = threadIdx.x % COLS, y = threadIdx.x / COLS;
  const int c = c0 + x;
  // kGateRows partial rows on: so many chunks, and so far in memory (past the last chunk of a batch row, over the other heads')
  const int dch = kGateRows % nchunk;
  const size_t step = ((size_t)(kGateRows / nchunk) * p.H * nchunk + dch) * G, over = (size_t)(p.H - 1) * nchunk * G;
  for (int row = y; row < kGateRows; row += R) {
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (c < G) {
      int ch = row % nchunk;
      size_t at = (((size_t)(row / nchunk) * p.H + h) * nchunk + ch) * G + c;
      for (int n = row; n < N; n += U * kGateRows) {
        float v[U];
#pragma unroll
        for (int i = 0; i < U; ++i) {
          v[i] = partial[n + i * kGateRows < N ? at : 0];
          v[i] = n + i * kGateRows < N ? v[i] : 0.0f;
          ch += dch;
          at += step;
          if (ch >= nchunk) {
            ch -= nchunk;
            at += over;
          }
        }
#pragma unroll
        for (int i = 0; i < U; ++i) acc[i & 3] += v[i];
      }
    }
    red[row][x] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  }
  for (int half = kGateRows / 2; half >= 1; half >>= 1) {
    __syncthreads();
    for (int row = y; row < half; row += R) red[row][x] += red[row + half][x];
  }
  if (y == 0 && c < G) {
    if (c < 2 * p.d) d_gate_w[(size_t)h * 2 * p.d + c] = red[0][x];
    else if (d_gate_b) d_gate_b[h] = red[0][x];
  }
}

}  // namespace blossom

#endif
