// Small kernels around the GEMMs: input packing, softmax cross-entropy with the per-worker 1/b_k, bias
// gradients and loss reduction.
#include <hip/hip_runtime.h>

#include "device_rows.h"
#include "dynb_internal.h"
#include "step_end.h"

namespace dynb {
namespace {

typedef __bf16 bf16;

template <typename T> __device__ inline T from_float(float v) { return (T)v; }

// Dense row -> worker.
__device__ inline int worker_of(const Segs& s, int row) {
  int k = 0;
  while (k + 1 < s.K && row >= s.off[k + 1]) ++k;
  return k;
}

__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ inline float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

// ---- pack: fp32 rows -> rows of T ---------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void pack_rows_kernel(const float* __restrict__ x, int D,
                                                        T* __restrict__ out, int64_t ld) {
  const int row = blockIdx.y;
  const float* src = x + (int64_t)row * D;
  T* dst = out + (int64_t)row * ld;
  for (int c = blockIdx.x * 256 + threadIdx.x; c < D; c += gridDim.x * 256)
    dst[c] = from_float<T>(src[c]);
}

// the same for rows whose length is a multiple of 8 with 16-byte aligned rows on both sides:
// 8 elements per lane (two 16-byte loads, one 16- or two 16-byte stores), grid-stride over all
// granules of the matrix
template <typename T>
__global__ __launch_bounds__(256) void pack_rows_vec_kernel(const float* __restrict__ x,
                                                            int64_t rows, int D,
                                                            T* __restrict__ out, int64_t ld) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  typedef T vec8T __attribute__((ext_vector_type(8)));
  const int gpr = D / 8;                       // granules per row
  const int64_t total = rows * gpr;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    const int64_t r = i / gpr;
    const int c = (int)(i - r * gpr) * 8;
    const f4 a = __builtin_nontemporal_load((const f4*)(x + r * D + c));
    const f4 b = __builtin_nontemporal_load((const f4*)(x + r * D + c + 4));
    const vec8T v = {from_float<T>(a[0]), from_float<T>(a[1]), from_float<T>(a[2]), from_float<T>(a[3]),
                     from_float<T>(b[0]), from_float<T>(b[1]), from_float<T>(b[2]), from_float<T>(b[3])};
    *(vec8T*)(out + r * ld + c) = v;
  }
}

// rows of at most 8 features (a pixel of few channels): one lane per row, one 16-byte store; the columns
// [D, 8) are written as zero, the rest of the padded row is never touched (it holds zeros)
__global__ __launch_bounds__(256) void pack_rows_narrow_kernel(const float* __restrict__ x,
                                                               int64_t rows, int D,
                                                               __bf16* __restrict__ out, int64_t ld) {
  typedef __bf16 vec8 __attribute__((ext_vector_type(8)));
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (r >= rows) return;
  vec8 v;
#pragma unroll
  for (int c = 0; c < 8; ++c) v[c] = c < D ? (__bf16)x[r * D + c] : (__bf16)0.f;
  *(vec8*)(out + r * ld) = v;
}

// ---- softmax cross-entropy, one wavefront per row -----------------------------------------
// dz = (softmax(z) - onehot(y)) / b_k for the rows of worker k; zero in the pad columns.
template <typename T>
__global__ __launch_bounds__(256) void softmax_xent_kernel(const float* __restrict__ z, int64_t ldz,
                                                           const int32_t* __restrict__ y, int C,
                                                           T* __restrict__ dz, int64_t ldd,
                                                           int ld_cols, float* __restrict__ rowloss,
                                                           Segs s) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= s.off[s.K]) return;
  const int k = worker_of(s, row);
  const int bk = s.off[k + 1] - s.off[k];
  T* drow = dz + (int64_t)row * ldd;
  const float* zr = z + (int64_t)row * ldz;
  int label = y[row];
  label = label < 0 ? 0 : (label >= C ? C - 1 : label);   // keeps the read in bounds
  if (ld_cols <= 1024 && (ldz & 3) == 0 && (ldd & 3) == 0) {
    // the whole row in registers: 16-byte loads, one exponential per element
    typedef T vec4T __attribute__((ext_vector_type(4)));
    float4 v[4];
    float m = -INFINITY;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c0 = 4 * (lane + 64 * u);
      v[u] = c0 < ld_cols ? *(const float4*)(zr + c0) : make_float4(0.f, 0.f, 0.f, 0.f);
      float* e = (float*)&v[u];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (c0 + q >= C) e[q] = -INFINITY;
        m = fmaxf(m, e[q]);
      }
    }
    m = wave_max(m);
    float sum = 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float* e = (float*)&v[u];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        e[q] = expf(e[q] - m);          // (exp(-inf) = 0 in the pad columns)
        sum += e[q];
      }
    }
    sum = wave_sum(sum);
    const float inv = 1.f / sum, scale = 1.f / (float)bk;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c0 = 4 * (lane + 64 * u);
      if (c0 >= ld_cols) continue;
      const float* e = (const float*)&v[u];
      vec4T o;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = c0 + q;
        o[q] = from_float<T>(c < C ? (e[q] * inv - (c == label ? 1.f : 0.f)) * scale : 0.f);
      }
      *(vec4T*)(drow + c0) = o;
    }
    if (lane == 0) rowloss[row] = logf(sum) - (zr[label] - m);
    return;
  }
  float m = -INFINITY;
  for (int c = lane; c < C; c += 64) m = fmaxf(m, zr[c]);
  m = wave_max(m);
  float sum = 0.f;
  for (int c = lane; c < C; c += 64) sum += expf(zr[c] - m);
  sum = wave_sum(sum);
  const float inv = 1.f / sum;
  const float scale = 1.f / (float)bk;
  for (int c = lane; c < ld_cols; c += 64) {
    float v = 0.f;
    if (c < C) v = (expf(zr[c] - m) * inv - (c == label ? 1.f : 0.f)) * scale;
    drow[c] = from_float<T>(v);
  }
  if (lane == 0) rowloss[row] = logf(sum) - (zr[label] - m);
}

// ---- the step's end (first K workgroups) and, behind them, the weighted aggregate, Eq. 2, of the small
// tensors listed in r -- one launch for what used to be two tiny ones ---------------------------------
// A workgroup takes 256 neighbouring elements of a range, a lane four of them; what bounds it is the way to
// memory and back, so the elements of four workers are in flight at once (one at a time, 49149 elements of 11
// workers: 11.9 us, 4.6 so).  Ascending k per element.
constexpr int RANGE_BLOCK = 256;
struct RangeBlocks {
  int first[MAX_RANGES + 1];               // first workgroup of every range
};

__global__ __launch_bounds__(64) void finalize_kernel(StepEnd end, Segs s, Lambdas lam, Ranges r, RangeBlocks rb) {
  if ((int)blockIdx.x < s.K) {
    end_worker(end, s, blockIdx.x);
    return;
  }
  const int block = blockIdx.x - s.K;
  int q = 0;                               // the last range whose first workgroup is not behind this one
  for (int step = 32; step > 0; step >>= 1)
    if (q + step < r.n && block >= rb.first[q + step]) q += step;
  const int64_t e0 = (int64_t)(block - rb.first[q]) * RANGE_BLOCK + threadIdx.x, n = r.len[q], off = r.off[q];
  const float* src[4];
  float acc[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {            // (lanes past the end repeat the last element)
    src[u] = end.grads + off + (e0 + 64 * u < n ? e0 + 64 * u : n - 1);
    acc[u] = 0.f;
  }
  int k = 0;
  for (; k + 4 <= lam.K; k += 4) {
    float v[4][4];
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
      for (int u = 0; u < 4; ++u) v[w][u] = src[u][(int64_t)(k + w) * end.P_pad];
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[u] += lam.w[k + w] * v[w][u];
  }
  for (; k < lam.K; ++k)
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[u] += lam.w[k] * src[u][(int64_t)k * end.P_pad];
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (e0 + 64 * u < n) end.out[off + e0 + 64 * u] = acc[u];
}

// ---- read and discard (see launch_touch) -------------------------------------------------
__global__ __launch_bounds__(256) void touch_kernel(const uint4* __restrict__ p, int64_t n,
                                                    uint32_t* sink) {
  uint32_t acc = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const uint4 v = p[i];
    acc |= v.x ^ v.y ^ v.z ^ v.w;
  }
  if (sink) *sink = acc;   // (sink is always null: the condition only keeps the loads alive)
}

// ---- sum of the split weight-gradient chunks, fixed order -------------------------------
__global__ __launch_bounds__(256) void wgrad_reduce_kernel(const float* __restrict__ partial,
                                                           int split, int64_t pstride, int64_t n,
                                                           float* __restrict__ out,
                                                           int64_t group_stride) {
  const int g = blockIdx.y;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256) {
    float acc = 0.f;
    for (int c = 0; c < split; ++c) acc += partial[((int64_t)g * split + c) * pstride + e];
    out[(int64_t)g * group_stride + e] = acc;
  }
}

inline int ok(const char* what) {
  return hipGetLastError() == hipSuccess ? DYNB_OK : fail(DYNB_ERR_HIP, "%s: launch failed", what);
}

}  // namespace

#define DISPATCH_T(dtype, CALL)                              \
  do {                                                       \
    if ((dtype) == DYNB_BF16) { typedef bf16 T; CALL; }      \
    else { typedef float T; CALL; }                          \
  } while (0)

int launch_pack_rows(int dtype, const float* x, int rows, int D, void* out, int64_t ld,
                     void* stream) {
  if (rows == 0) return DYNB_OK;
  const int es = dtype == DYNB_BF16 ? 2 : 4;
  Timed t(KC_PACK, stream, 0, (double)rows * D * (4 + es));
  if ((D & 7) == 0 && (ld & 7) == 0 && !(((uintptr_t)x | (uintptr_t)out) & 31)) {
    int64_t blocks = ((int64_t)rows * (D / 8) + 255) / 256;
    if (blocks > 256 * 32) blocks = 256 * 32;
    DISPATCH_T(dtype, hipLaunchKernelGGL(pack_rows_vec_kernel<T>, dim3((unsigned)blocks), dim3(256), 0,
                                         (hipStream_t)stream, x, (int64_t)rows, D, (T*)out, ld));
    return ok("pack_rows");
  }
  if (dtype == DYNB_BF16 && D <= 8 && (ld & 7) == 0 && !((uintptr_t)out & 15)) {
    hipLaunchKernelGGL(pack_rows_narrow_kernel, dim3((unsigned)((rows + 255) / 256)), dim3(256), 0,
                       (hipStream_t)stream, x, (int64_t)rows, D, (__bf16*)out, ld);
    return ok("pack_rows");
  }
  dim3 grid((D + 255) / 256 > 8 ? 8 : (D + 255) / 256, rows);
  DISPATCH_T(dtype, hipLaunchKernelGGL(pack_rows_kernel<T>, grid, dim3(256), 0,
                                       (hipStream_t)stream, x, D, (T*)out, ld));
  return ok("pack_rows");
}

int launch_softmax_xent(int dtype, const float* logits, int64_t ldz, const int32_t* y, int C,
                        void* dz, int64_t ldd, int ld_cols, float* rowloss, const Segs& s,
                        void* stream) {
  const int rows = s.off[s.K];
  if (rows == 0) return DYNB_OK;
  Timed t(KC_SOFTMAX, stream, 0, (double)rows * C * 6);
  DISPATCH_T(dtype, hipLaunchKernelGGL(softmax_xent_kernel<T>, dim3((rows + 3) / 4), dim3(256), 0,
                                       (hipStream_t)stream, logits, ldz, y, C, (T*)dz, ldd,
                                       ld_cols, rowloss, s));
  return ok("softmax_xent");
}

// Bias gradient from the row-major gradient dy [rows][ld] (bf16): one workgroup per (64 features,
// worker); 8 lanes cover the 128 bytes of a row, 32 row-lanes walk the worker's rows, the
// partial sums meet in a fixed order.
__global__ __launch_bounds__(256) void bias_grad_rows_kernel(const bf16* __restrict__ dy, int64_t ld,
                                                             int N, float* __restrict__ grads,
                                                             int64_t group_stride, Segs s) {
  __shared__ float red[4][64];
  const int cg = threadIdx.x & 7, rl = threadIdx.x >> 3;
  const int c0 = blockIdx.x * 64 + cg * 8, k = blockIdx.y;
  const int r0 = s.off[k], n = s.off[k + 1] - r0;
  float acc[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) acc[j] = 0.f;
  for (int r = rl; r < n; r += 32) {
    float v[8];
    unpack8(load8(dy + (int64_t)(r0 + r) * ld + c0), v);
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] += v[j];
  }
  sum_over_rows<8>(acc, red);
  if (rl == 0) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (c0 + j < N) grads[(int64_t)k * group_stride + c0 + j] = acc[j];
  }
}

int launch_bias_grad_rows(const void* dy, int64_t ld, int N, float* grads, int64_t group_stride,
                          const Segs& s, void* stream) {
  if (N == 0) return DYNB_OK;
  if (ld % 64 || ld < N) return fail(DYNB_ERR_BADARG, "bias_grad_rows: the row pitch must cover whole 64-feature blocks");
  Timed t(KC_BIAS_GRAD, stream, 0, (double)s.off[s.K] * N * 2);
  hipLaunchKernelGGL(bias_grad_rows_kernel, dim3((unsigned)(ld / 64), s.K), dim3(256), 0,
                     (hipStream_t)stream, (const bf16*)dy, ld, N, grads, group_stride, s);
  return ok("bias_grad_rows");
}

int launch_touch(const void* p, int64_t bytes, void* stream) {
  if (bytes < 16) return DYNB_OK;
  Timed t(KC_PACK, stream, 0, (double)bytes);   // (counted with the other staging passes)
  int64_t bx = (bytes / 16 + 255) / 256;
  if (bx > 2048) bx = 2048;
  hipLaunchKernelGGL(touch_kernel, dim3((unsigned)bx), dim3(256), 0, (hipStream_t)stream,
                     (const uint4*)p, bytes / 16, (uint32_t*)nullptr);
  return ok("touch");
}

int launch_finalize(const StepEnd& end, const Segs& s, const Lambdas* lam, const Ranges* small, void* stream) {
  Lambdas l;
  l.K = 0;
  Ranges r;
  r.n = 0;
  RangeBlocks rb;
  int64_t total = 0, blocks = 0;
  if (end.out && lam && small) {
    l = *lam;
    r = *small;
    for (int i = 0; i < r.n; ++i) {
      rb.first[i] = (int)blocks;
      blocks += (r.len[i] + RANGE_BLOCK - 1) / RANGE_BLOCK;
      total += r.len[i];
    }
  }
  for (int i = r.n; i <= MAX_RANGES; ++i) rb.first[i] = (int)blocks;
  if (blocks >= ((int64_t)1 << 31) - DYNB_MAX_WORKERS) return fail(DYNB_ERR_UNSUPPORTED, "finalize: ranges too long for one launch");
  Timed t(KC_FINALIZE, stream, 2.0 * l.K * total, 4.0 * (l.K + 1) * total);
  hipLaunchKernelGGL(finalize_kernel, dim3((unsigned)(s.K + blocks)), dim3(64), 0, (hipStream_t)stream, end, s, l, r, rb);
  return ok("finalize");
}

int launch_wgrad_reduce(const float* partial, int split, int64_t partial_stride, int64_t n,
                        float* out, int64_t group_stride, int K, void* stream) {
  Timed t(KC_GEMM_WGRAD, stream, 0, 0);
  int64_t bx = (n + 255) / 256;
  if (bx > 1024) bx = 1024;
  hipLaunchKernelGGL(wgrad_reduce_kernel, dim3((unsigned)bx, K), dim3(256), 0, (hipStream_t)stream,
                     partial, split, partial_stride, n, out, group_stride);
  return ok("wgrad_reduce");
}

}  // namespace dynb
