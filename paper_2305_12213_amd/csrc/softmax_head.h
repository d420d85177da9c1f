// Softmax cross-entropy behind the last product of a model, by the workgroup that holds whole rows of
// logits: shared by the fp32 and the bf16 kernel.
#ifndef DYNB_SOFTMAX_HEAD_H
#define DYNB_SOFTMAX_HEAD_H

#include <hip/hip_runtime.h>

#include "dynb_internal.h"

namespace dynb {

struct NoHead {};

// Rows of the worker that owns `row` (uniform loads, one compare per worker and lane).
__device__ inline int rows_of_owner(const Segs& s, int row) {
  int n = 1;
  for (int k = 0; k < s.K; ++k) {
    const int a = s.off[k], b = s.off[k + 1];
    if (row >= a && row < b) n = b - a;
  }
  return n;
}

// One row on `lanes` (a power of two) neighbouring lanes, four logits e[] each from column c0 on: e becomes
// (softmax - onehot(label)) / rows, zero from column C on; returns the row's loss.  The additions are
// those of softmax_xent_kernel.
__device__ inline float softmax_row(int lanes, float (&e)[4], int c0, int C, int label, float label_logit, int rows) {
  float m = -INFINITY;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (c0 + q >= C) e[q] = -INFINITY;
    m = fmaxf(m, e[q]);
  }
  for (int o = lanes / 2; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
  float sum = 0.f;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    e[q] = expf(e[q] - m);
    sum += e[q];
  }
  for (int o = lanes / 2; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
  const float inv = 1.f / sum, scale = 1.f / (float)rows;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int c = c0 + q;
    e[q] = c < C ? (e[q] * inv - (c == label ? 1.f : 0.f)) * scale : 0.f;
  }
  return logf(sum) - (label_logit - m);
}

}  // namespace dynb

#endif
