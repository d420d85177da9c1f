// Kernels around the implicit-GEMM convolutions (NHWC, 3x3, zero padding 1; bf16 storage):
// global average pooling forward/backward.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_rows.h"
#include "dynb_internal.h"

namespace dynb {
namespace {

// pooled[n][c] = mean over the HW pixels of act[(n, pixel)][c]   (fp32 sum in a fixed order,
// bf16 store).  One workgroup per (sample, 8 LPR channels); padding channels are written as zero (those
// beyond act's pitch hold zeros and keep them).
// (eight rows of a lane in flight: 512 x 32 x 32 x 64 19 -> 12.8 us, 167 x 28 x 28 x 24 10.8 -> 5.8.  Of the last 128
// pixels only as many as there are: always eight, a lane's own and seven times the last one, took 2048 x 2 x 2 x 512
// from 23 us, with one, to 28; now 14.  2048 x 7 x 7 x 128 10.0 -> 6.8.)
template <int LPR>
__global__ __launch_bounds__(32 * LPR) void gap_forward_kernel(const bf16* __restrict__ act, int64_t lda,
                                                          int HW, int C, bf16* __restrict__ pooled,
                                                          int64_t ldp) {
  __shared__ float red[4][8 * LPR];
  const int cg = threadIdx.x % LPR, rl = threadIdx.x / LPR;
  const int n = blockIdx.x, c0 = blockIdx.y * (8 * LPR) + cg * 8;
  const bf16* base = act + (int64_t)n * HW * lda + blockIdx.y * (8 * LPR);
  float acc[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) acc[j] = 0.f;
  auto take = [&](auto rows, int p0) {
    constexpr int F = decltype(rows)::value;
    uint4 q[F];
    load_rows<LPR>(base + (int64_t)p0 * lda, lda, HW - p0, q);
#pragma unroll
    for (int i = 0; i < F; ++i) {
      float v[8];
      unpack8(q[i], v);
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[j] += p0 + rl + 32 * i < HW ? v[j] : 0.f;
    }
  };
  int p0 = 0;
  for (; HW - p0 > 16 * ROWS_IN_FLIGHT; p0 += 32 * ROWS_IN_FLIGHT) take(std::integral_constant<int, ROWS_IN_FLIGHT>(), p0);
  if (HW - p0 > 64) take(std::integral_constant<int, 4>(), p0);
  else if (HW - p0 > 32) take(std::integral_constant<int, 2>(), p0);
  else if (HW - p0 > 0) take(std::integral_constant<int, 1>(), p0);
  sum_over_rows<LPR>(acc, red);
  if (rl == 0) {
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = c0 + j < C ? acc[j] / (float)HW : 0.f;
    store8(pooled + (int64_t)n * ldp + c0, pack8(acc));
  }
}

// d act[(n, pixel)][c] = d pooled[n][c] / HW, masked by act > 0 when the pooled layer's producer
// applied a ReLU.  One lane per 8 channels of a row; `gpr` = 16-byte granules per row.
__global__ __launch_bounds__(256) void gap_backward_kernel(const bf16* __restrict__ dpooled,
                                                           int64_t ldp, const bf16* __restrict__ act,
                                                           int64_t lda, int HW, int gpr, int64_t total,
                                                           int relu, bf16* __restrict__ dact,
                                                           int64_t ldd) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const int64_t row = i / gpr;   // (n, pixel)
  const int c0 = (int)(i - row * gpr) * 8;
  float v[8];
  unpack8(load8(dpooled + (row / HW) * ldp + c0), v);
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j] = v[j] / (float)HW;
  if (relu) {
    float a[8];
    unpack8(load8(act + row * lda + c0), a);
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (!(a[j] > 0.f)) v[j] = 0.f;
  }
  store8(dact + row * ldd + c0, pack8(v));
}

inline int ok(const char* what) {
  return hipGetLastError() == hipSuccess ? DYNB_OK : fail(DYNB_ERR_HIP, "%s: launch failed", what);
}

}  // namespace

int launch_gap_forward(const void* act, int64_t lda, int HW, int C, int samples, void* pooled,
                       int64_t ldp, void* stream) {
  if (samples == 0) return DYNB_OK;
  const bool narrow = lda == NARROW_PITCH;
  if ((lda % 64 && !narrow) || ldp % 64 || ldp < C || lda < C)
    return fail(DYNB_ERR_BADARG, "gap_forward: bad pitches");
  Timed t(KC_CONV_AUX, stream, 0, (double)samples * HW * C * 2);
  const hipStream_t st = (hipStream_t)stream;
  if (narrow)
    hipLaunchKernelGGL(gap_forward_kernel<4>, dim3(samples), dim3(128), 0, st, (const bf16*)act, lda, HW, C,
                       (bf16*)pooled, ldp);
  else
    hipLaunchKernelGGL(gap_forward_kernel<8>, dim3(samples, (C + 63) / 64), dim3(256), 0, st, (const bf16*)act, lda,
                       HW, C, (bf16*)pooled, ldp);
  return ok("gap_forward");
}

int launch_gap_backward(const void* dpooled, int64_t ldp, const void* act, int64_t lda, int HW,
                        int C, int samples, int relu, void* dact, int64_t ldd, void* stream) {
  if (samples == 0) return DYNB_OK;
  if (lda % 8 || ldp % 8 || ldd % 8 || ldp < ldd || lda < ldd)
    return fail(DYNB_ERR_BADARG, "gap_backward: bad pitches");
  const int gpr = (int)(ldd / 8);
  const int64_t total = (int64_t)samples * HW * gpr;
  Timed t(KC_CONV_AUX, stream, 0, (double)samples * HW * C * 4);
  hipLaunchKernelGGL(gap_backward_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0,
                     (hipStream_t)stream, (const bf16*)dpooled, ldp, (const bf16*)act, lda, HW, gpr,
                     total, relu, (bf16*)dact, ldd);
  return ok("gap_backward");
}

}  // namespace dynb
