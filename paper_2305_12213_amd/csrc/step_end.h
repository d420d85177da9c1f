// What ends an iteration besides the gradients: a worker's mean loss and the zero padding of its
// gradient vector.  Shared by the launches that can take it along.
#ifndef DYNB_STEP_END_H
#define DYNB_STEP_END_H

#include <hip/hip_runtime.h>

#include "dynb_internal.h"

namespace dynb {

// Worker g, by the first wave of a workgroup.
__device__ inline void end_worker(const StepEnd& e, const Segs& s, int g) {
  const int lane = threadIdx.x;
  const int r0 = s.off[g], bk = s.off[g + 1] - r0;
  // eight independent partial sums per lane: the loads of a round are in flight together
  float part[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int i = lane; i < bk; i += 512) {
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (i + 64 * u < bk) part[u] += e.rowloss[r0 + i + 64 * u];
  }
  float acc = ((part[0] + part[1]) + (part[2] + part[3])) + ((part[4] + part[5]) + (part[6] + part[7]));
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if (lane == 0) e.loss[g] = bk > 0 ? acc / (float)bk : 0.f;
  for (int64_t p = e.P + lane; p < e.P_pad; p += 64) e.grads[(int64_t)g * e.P_pad + p] = 0.f;
  // (the aggregate's padding is written here, not summed from the tails above: workgroups of
  // one launch run in no particular order)
  if (e.out && g == 0)
    for (int64_t p = e.P + lane; p < e.P_pad; p += 64) e.out[p] = 0.f;
}

}  // namespace dynb

#endif
