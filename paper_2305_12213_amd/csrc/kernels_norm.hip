// Batch normalisation over each worker's own rows and residual additions (bf16 storage).
// A "row" is a sample or a pixel; worker k owns rows [off_k, off_{k+1}).  The statistics of a
// worker never see another worker's rows, so every reduction here runs per (worker, channel).
// The rows of a worker are cut into chunks of CHUNK_ROWS; one workgroup takes one chunk and 8 LPR = 64 or 32
// channels (a lane: 8 channels of a row = one 16-byte access, LPR lanes = the 128 or 64 bytes of a row,
// 32 rows per pass), writes the chunk's partial result, and a second small kernel merges the
// chunks of each worker in a fixed order.  All sums are fp32 and deterministic.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_rows.h"
#include "dynb_internal.h"

namespace dynb {
namespace {

constexpr int CHUNK_ROWS = BN_CHUNK_ROWS;
constexpr int PASSES = CHUNK_ROWS / 32;   // rows per lane
static_assert(PASSES == ROWS_IN_FLIGHT, "a chunk is fetched at once");

// first[k] = index of worker k's first chunk; first[K] = number of chunks
struct Chunks {
  int first[DYNB_MAX_WORKERS + 1];
};

// worker, first row and row count (at least one) of a chunk < first[K]: the last worker whose first chunk
// is not behind it (a bisection: each step is a dependent scalar load)
__device__ inline void chunk_span(const Segs& s, const Chunks& ch, int chunk, int& k, int& r0, int& n) {
  k = 0;
  for (int step = DYNB_MAX_WORKERS / 2; step > 0; step >>= 1)
    if (k + step < s.K && chunk >= ch.first[k + step]) k += step;
  r0 = s.off[k] + (chunk - ch.first[k]) * CHUNK_ROWS;
  n = min(CHUNK_ROWS, s.off[k + 1] - r0);
}

// Which of four per-channel arrays this thread fetches (8 LPR threads each; whole waves where that is one).
template <int LPR>
__device__ inline int array_of() {
  const int a = threadIdx.x / (8 * LPR);
  return LPR == 8 ? __builtin_amdgcn_readfirstlane(a) : a;
}

// Mean and sum of centred squares of one chunk (its values stay in registers between the two).
template <int LPR>
__global__ __launch_bounds__(32 * LPR) void bn_chunk_stats_kernel(const bf16* __restrict__ x, int64_t ld,
                                                             int C, float* __restrict__ pmean,
                                                             float* __restrict__ pm2, Segs s, Chunks ch) {
  __shared__ float red[4][8 * LPR];
  const int rl = threadIdx.x / LPR, chunk = blockIdx.x, c0 = blockIdx.y * (8 * LPR);
  int k, r0, n;
  chunk_span(s, ch, chunk, k, r0, n);
  uint4 q[PASSES];
  load_rows<LPR>(x + (int64_t)r0 * ld + c0, ld, n, q);
  float acc[8], mu[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) acc[j] = 0.f;
#pragma unroll
  for (int i = 0; i < PASSES; ++i) {
    float v[8];
    unpack8(q[i], v);
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] += rl + 32 * i < n ? v[j] : 0.f;
  }
  sum_over_rows<LPR>(acc, red);
  const int l = threadIdx.x % (8 * LPR);
  const float mean = (((red[0][l] + red[1][l]) + red[2][l]) + red[3][l]) / (float)n;
#pragma unroll
  for (int j = 0; j < 8; ++j) { mu[j] = acc[j] / (float)n; acc[j] = 0.f; }
#pragma unroll
  for (int i = 0; i < PASSES; ++i) {
    if (rl + 32 * i < n) {
      float v[8];
      unpack8(q[i], v);
#pragma unroll
      for (int j = 0; j < 8; ++j) { const float d = v[j] - mu[j]; acc[j] += d * d; }
    }
  }
  const float m2 = channel_sum<LPR>(acc, red);
  if (threadIdx.x < 8 * LPR && c0 + l < C) {
    pmean[(int64_t)chunk * C + c0 + l] = mean;
    pm2[(int64_t)chunk * C + c0 + l] = m2;
  }
}

// Sum over the chunks of one worker, for 16 channels at a time: 1024 threads = 16 waves of 16 channels
// x 4 lanes.  Wave q adds the terms of chunks q, q+16, ...: lane u of it those of every fourth of them
// (while whole groups of four are left; the rest goes to lane 0), the four lanes are then added in
// pairs, the 16 waves in ascending order.  term(j) = value of chunk j for this thread's channel.  Every
// thread of the channel gets the total.  What bounds a merge is the chain of loads of one lane: 64
// channels x 16 lanes per workgroup, with these four sums in one lane, took 9.4 us for 556 chunks,
// this split (the same additions) 6.5.
constexpr int MERGE_C = 16;
template <typename F>
__device__ inline float sum_over_chunks(int nc, float (*red)[MERGE_C], F term) {
  const int q = threadIdx.x >> 6, u = (threadIdx.x >> 4) & 3, cl = threadIdx.x & 15;
  float a = 0.f;
  int j = q;
  for (; j + 48 + 7 * 64 < nc; j += 8 * 64) {   // (eight loads in flight, then added in order)
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = term(j + 64 * i + 16 * u);
#pragma unroll
    for (int i = 0; i < 8; ++i) a += v[i];
  }
  for (; j + 48 < nc; j += 64) a += term(j + 16 * u);
  if (u == 0)
    for (; j < nc; j += 16) a += term(j);
  a += __shfl_xor(a, 16);
  a += __shfl_xor(a, 32);
  __syncthreads();
  if (u == 0) red[q][cl] = a;
  __syncthreads();
  float t = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) t += red[i][cl];
  return t;
}

// mean[k][c], rstd[k][c] from the chunk moments of worker k: the mean is the weighted sum of
// the chunk means, the sum of squares follows from the parallel-axis relation
//   M2 = sum_j (M2_j + n_j (mean_j - mean)^2)
// -- two plain sums in a fixed order.
__global__ __launch_bounds__(1024) void bn_merge_stats_kernel(const float* __restrict__ pmean,
                                                              const float* __restrict__ pm2, int C,
                                                              float eps, float* __restrict__ mean,
                                                              float* __restrict__ rstd, Segs s, Chunks ch) {
  __shared__ float red[16][MERGE_C];
  const int c = blockIdx.x * MERGE_C + (threadIdx.x & 15), k = blockIdx.y;
  const int rows = s.off[k + 1] - s.off[k];
  if (rows <= 0) return;                      // (uniform over the workgroup)
  const int first = ch.first[k], nc = ch.first[k + 1] - first;
  const int cc = c < C ? c : C - 1;           // lanes past the last channel repeat it, unused
  const float n = (float)rows;
  auto rows_of = [&](int j) { return (float)min(CHUNK_ROWS, rows - j * CHUNK_ROWS); };
  const float mu = sum_over_chunks(nc, red, [&](int j) {
                     return rows_of(j) * pmean[(int64_t)(first + j) * C + cc];
                   }) / n;
  const float m2 = sum_over_chunks(nc, red, [&](int j) {
    const float d = pmean[(int64_t)(first + j) * C + cc] - mu;
    return pm2[(int64_t)(first + j) * C + cc] + rows_of(j) * d * d;
  });
  if (threadIdx.x < MERGE_C && c < C) {
    mean[(int64_t)k * C + c] = mu;
    rstd[(int64_t)k * C + c] = 1.f / sqrtf(m2 / n + eps);
  }
}

// y = relu?(gamma * ((x - mean_k) * rstd_k) + beta); padding channels are written as zero.
// With SKIP, the residual addition behind the normalisation is applied in the same pass:
// y = relu_sum?(bf16(normalised) + skip) -- rounded as if the normalised tensor had been stored.
// What bounds these element-wise passes is the bytes in flight: a lane handles eight rows, asks for all of
// them at once, and meanwhile each of the 64 x 4 coefficients is fetched by one lane and handed on in LDS.
// 524288 rows of 64 channels (67 MB a tensor), against every lane fetching its own 32 coefficients and rows
// one by one behind a branch: this pass 27 -> 22 us, with the addition 44 -> 33, input gradient 39 -> 32,
// parameter gradients 31 -> 22 (6.0 - 6.3 TB/s each), statistics 14.3 -> 13.1.
template <int LPR, bool SKIP>
__global__ __launch_bounds__(32 * LPR) void bn_apply_kernel(const bf16* __restrict__ x, int64_t ldx, int C,
                                                       const float* __restrict__ gamma,
                                                       const float* __restrict__ beta,
                                                       const float* __restrict__ mean,
                                                       const float* __restrict__ rstd, int relu,
                                                       const bf16* __restrict__ skip, int64_t lds_,
                                                       int relu_sum, bf16* __restrict__ y, int64_t ldy,
                                                       Segs s, Chunks ch) {
  __shared__ __align__(16) float coef[4][8 * LPR];              // mean, rstd, gamma, beta
  const int rl = threadIdx.x / LPR, cg = threadIdx.x % LPR, c0 = blockIdx.y * (8 * LPR);
  int k, r0, n;
  chunk_span(s, ch, blockIdx.x, k, r0, n);
  const int what = array_of<LPR>(), c = c0 + threadIdx.x % (8 * LPR);
  const float* const from = what == 0 ? mean + (int64_t)k * C : what == 1 ? rstd + (int64_t)k * C
                            : what == 2 ? gamma : beta;
  const float mine = from[c < C ? c : C - 1];
  uint4 q[PASSES], z[PASSES];
  load_rows<LPR>(x + (int64_t)r0 * ldx + c0, ldx, n, q);
  if (SKIP) load_rows<LPR>(skip + (int64_t)r0 * lds_ + c0, lds_, n, z);
  coef[what][threadIdx.x % (8 * LPR)] = c < C ? mine : 0.f;       // (padding channels: all zero, whatever x holds
  __syncthreads();                                         // there -- see keep below)
  float mu[8], rs[8], ga[8], be[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    mu[j] = coef[0][cg * 8 + j]; rs[j] = coef[1][cg * 8 + j];
    ga[j] = coef[2][cg * 8 + j]; be[j] = coef[3][cg * 8 + j];
  }
  const uint4 keep = keep8(C - c0 - cg * 8);
  bf16* const yb = y + (int64_t)r0 * ldy + c0 + cg * 8;
#pragma unroll
  for (int i = 0; i < PASSES; ++i) {
    const int r = rl + 32 * i;
    if (r < n) {
      float v[8];
      unpack8(q[i], v);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        v[j] = ga[j] * ((v[j] - mu[j]) * rs[j]) + be[j];
        if (relu) v[j] = fmaxf(v[j], 0.f);
      }
      uint4 o = pack8(v) & keep;
      if (SKIP) {
        float w[8];
        unpack8(o, v);                           // the normalised values as they would be stored
        unpack8(z[i], w);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          v[j] += w[j];
          if (relu_sum) v[j] = fmaxf(v[j], 0.f);
        }
        o = pack8(v);
      }
      store8(yb + (int64_t)r * ldy, o);
    }
  }
}

// Chunk sums of dy and of dy * xhat (dy already carries this layer's ReLU mask).
template <int LPR>
__global__ __launch_bounds__(32 * LPR) void bn_chunk_param_grad_kernel(
    const bf16* __restrict__ dy, int64_t ldd, const bf16* __restrict__ x, int64_t ldx, int C,
    const float* __restrict__ mean, const float* __restrict__ rstd, float* __restrict__ pdg,
    float* __restrict__ pdb, Segs s, Chunks ch) {
  __shared__ __align__(16) float coef[2][8 * LPR];              // mean, rstd
  __shared__ float red[2][4][8 * LPR];
  const int rl = threadIdx.x / LPR, cg = threadIdx.x % LPR, chunk = blockIdx.x, c0 = blockIdx.y * (8 * LPR);
  int k, r0, n;
  chunk_span(s, ch, chunk, k, r0, n);
  const int what = array_of<LPR>(), c = c0 + threadIdx.x % (8 * LPR);
  const float mine = (what == 0 ? mean : rstd)[(int64_t)k * C + (c < C ? c : C - 1)];
  uint4 q[PASSES], z[PASSES];
  load_rows<LPR>(x + (int64_t)r0 * ldx + c0, ldx, n, q);
  load_rows<LPR>(dy + (int64_t)r0 * ldd + c0, ldd, n, z);
  if (what < 2) coef[what][threadIdx.x % (8 * LPR)] = c < C ? mine : 0.f;
  __syncthreads();
  float mu[8], rs[8], ag[8], ab[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    mu[j] = coef[0][cg * 8 + j]; rs[j] = coef[1][cg * 8 + j];
    ag[j] = 0.f; ab[j] = 0.f;
  }
#pragma unroll
  for (int i = 0; i < PASSES; ++i) {
    if (rl + 32 * i < n) {
      float v[8], d[8];
      unpack8(q[i], v);
      unpack8(z[i], d);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        ab[j] += d[j];
        ag[j] += d[j] * ((v[j] - mu[j]) * rs[j]);
      }
    }
  }
  sum_over_row_group<LPR>(ag, red[0]);
  sum_over_row_group<LPR>(ab, red[1]);
  __syncthreads();
  if (what < 2 && c < C) {
    const float(*const t)[8 * LPR] = red[what];
    const int l = threadIdx.x % (8 * LPR);
    (what == 0 ? pdg : pdb)[(int64_t)chunk * C + c] = ((t[0][l] + t[1][l]) + t[2][l]) + t[3][l];
  }
}

// dgamma[k][c], dbeta[k][c] = the chunk sums of worker k added in a fixed order, written into
// worker k's gradient vector; a worker without rows gets zeros.
__global__ __launch_bounds__(1024) void bn_merge_param_grad_kernel(const float* __restrict__ pdg,
                                                                   const float* __restrict__ pdb, int C,
                                                                   float* __restrict__ dgamma,
                                                                   float* __restrict__ dbeta,
                                                                   int64_t group_stride, Chunks ch) {
  __shared__ float red[16][MERGE_C];
  const int c = blockIdx.x * MERGE_C + (threadIdx.x & 15), k = blockIdx.y;
  const int first = ch.first[k], nc = ch.first[k + 1] - first;
  const int cc = c < C ? c : C - 1;
  const float g = sum_over_chunks(nc, red, [&](int j) { return pdg[(int64_t)(first + j) * C + cc]; });
  const float b = sum_over_chunks(nc, red, [&](int j) { return pdb[(int64_t)(first + j) * C + cc]; });
  if (threadIdx.x < MERGE_C && c < C) {
    dgamma[(int64_t)k * group_stride + c] = g;
    dbeta[(int64_t)k * group_stride + c] = b;
  }
}

// dx = gamma * rstd * (dy - dbeta/n - xhat * dgamma/n), masked by the producer's ReLU (x > 0);
// padding channels are written as zero
template <int LPR>
__global__ __launch_bounds__(32 * LPR) void bn_input_grad_kernel(
    const bf16* __restrict__ dy, int64_t ldd, const bf16* __restrict__ x, int64_t ldx, int C,
    const float* __restrict__ gamma, const float* __restrict__ mean, const float* __restrict__ rstd,
    const float* __restrict__ dgamma, const float* __restrict__ dbeta, int64_t group_stride,
    int relu_below, bf16* __restrict__ dx, int64_t ldo, Segs s, Chunks ch) {
  __shared__ __align__(16) float coef[5][8 * LPR];              // mean, rstd, dgamma / n, dbeta / n, gamma rstd
  const int rl = threadIdx.x / LPR, cg = threadIdx.x % LPR, c0 = blockIdx.y * (8 * LPR);
  int k, r0, n;
  chunk_span(s, ch, blockIdx.x, k, r0, n);
  const int what = array_of<LPR>(), l = threadIdx.x % (8 * LPR), c = c0 + l;
  const float* const from = what == 0   ? mean + (int64_t)k * C
                            : what == 1 ? rstd + (int64_t)k * C
                            : what == 2 ? dgamma + (int64_t)k * group_stride
                                        : dbeta + (int64_t)k * group_stride;
  const float mine = from[c < C ? c : C - 1], ga = gamma[c < C ? c : C - 1];
  uint4 q[PASSES], z[PASSES];
  load_rows<LPR>(x + (int64_t)r0 * ldx + c0, ldx, n, q);
  load_rows<LPR>(dy + (int64_t)r0 * ldd + c0, ldd, n, z);
  const float rows = (float)(s.off[k + 1] - s.off[k]);
  coef[what][l] = c < C ? (what < 2 ? mine : mine / rows) : 0.f;
  if (what == 1) coef[4][l] = c < C ? ga * mine : 0.f;
  __syncthreads();
  float mu[8], rs[8], gr[8], mg[8], mb[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    mu[j] = coef[0][cg * 8 + j]; rs[j] = coef[1][cg * 8 + j];
    mg[j] = coef[2][cg * 8 + j]; mb[j] = coef[3][cg * 8 + j]; gr[j] = coef[4][cg * 8 + j];
  }
  const uint4 keep = keep8(C - c0 - cg * 8);
  bf16* const ob = dx + (int64_t)r0 * ldo + c0 + cg * 8;
#pragma unroll
  for (int i = 0; i < PASSES; ++i) {
    const int r = rl + 32 * i;
    if (r < n) {
      float v[8], d[8];
      unpack8(q[i], v);
      unpack8(z[i], d);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        d[j] = gr[j] * (d[j] - mb[j] - ((v[j] - mu[j]) * rs[j]) * mg[j]);
        if (relu_below && !(v[j] > 0.f)) d[j] = 0.f;
      }
      store8(ob + (int64_t)r * ldo, pack8(d) & keep);
    }
  }
}

// Element-wise kernels: one lane takes 8 channels of a row; `gpr` = 16-byte granules per row
// (the padded width / 8; padding channels hold zeros on both sides).

// out = relu?(a + b)
__global__ __launch_bounds__(256) void add_forward_kernel(const bf16* __restrict__ a, int64_t lda,
                                                          const bf16* __restrict__ b, int64_t ldb,
                                                          int gpr, int64_t total, int relu,
                                                          bf16* __restrict__ out, int64_t ldo) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const int64_t row = i / gpr;
  const int c0 = (int)(i - row * gpr) * 8;
  float u[8], v[8];
  unpack8(load8(a + row * lda + c0), u);
  unpack8(load8(b + row * ldb + c0), v);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    u[j] += v[j];
    if (relu) u[j] = fmaxf(u[j], 0.f);
  }
  store8(out + row * ldo + c0, pack8(u));
}

// dst = (accumulate ? dst : 0) + src, masked by act > 0 when `relu` (act = the stored output of
// the layer whose gradient dst is)
__global__ __launch_bounds__(256) void grad_route_kernel(const bf16* __restrict__ src, int64_t lds_,
                                                         const bf16* __restrict__ act, int64_t lda,
                                                         int gpr, int64_t total, int relu,
                                                         int accumulate, bf16* __restrict__ dst,
                                                         int64_t ldd) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const int64_t row = i / gpr;
  const int c0 = (int)(i - row * gpr) * 8;
  float v[8];
  unpack8(load8(src + row * lds_ + c0), v);
  if (relu) {
    float a[8];
    unpack8(load8(act + row * lda + c0), a);
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (!(a[j] > 0.f)) v[j] = 0.f;
  }
  if (accumulate) {
    float d[8];
    unpack8(load8(dst + row * ldd + c0), d);
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] += d[j];
  }
  store8(dst + row * ldd + c0, pack8(v));
}

inline int ok(const char* what) {
  return hipGetLastError() == hipSuccess ? DYNB_OK : fail(DYNB_ERR_HIP, "%s: launch failed", what);
}

Chunks make_chunks(const Segs& s) {
  Chunks ch;
  ch.first[0] = 0;
  for (int k = 0; k < s.K; ++k)
    ch.first[k + 1] = ch.first[k] + (s.off[k + 1] - s.off[k] + CHUNK_ROWS - 1) / CHUNK_ROWS;
  for (int k = s.K + 1; k <= DYNB_MAX_WORKERS; ++k) ch.first[k] = ch.first[s.K];
  return ch;
}

}  // namespace

int launch_bn_forward(const void* x, int64_t ldx, int C, const float* gamma, const float* beta,
                      float eps, int relu, float* mean, float* rstd, float* scratch,
                      const void* skip, int64_t lds_, int relu_sum, void* y, int64_t ldy,
                      const Segs& s, void* stream) {
  const int rows = s.off[s.K];
  if (rows == 0 || C == 0) return DYNB_OK;
  const Chunks ch = make_chunks(s);
  const int nch = ch.first[s.K];
  float* pmean = scratch;
  float* pm2 = scratch + (int64_t)nch * C;
  // algorithmic bytes: x read and y written once (+ the skip tensor); the statistics pass reads x again
  Timed t(KC_NORM, stream, 0, (double)rows * C * (skip ? 6 : 4));
  const hipStream_t st = (hipStream_t)stream;
  auto launch = [&](auto lpr) {
    constexpr int LPR = decltype(lpr)::value, COLS = 8 * LPR;
    hipLaunchKernelGGL(bn_chunk_stats_kernel<LPR>, dim3(nch, (C + COLS - 1) / COLS), dim3(32 * LPR), 0, st,
                       (const bf16*)x, ldx, C, pmean, pm2, s, ch);
    hipLaunchKernelGGL(bn_merge_stats_kernel, dim3((C + MERGE_C - 1) / MERGE_C, s.K), dim3(1024), 0, st, pmean,
                       pm2, C, eps, mean, rstd, s, ch);
    const auto apply = skip ? bn_apply_kernel<LPR, true> : bn_apply_kernel<LPR, false>;
    hipLaunchKernelGGL(apply, dim3(nch, (unsigned)(ldy / COLS)), dim3(32 * LPR), 0, st, (const bf16*)x, ldx, C,
                       gamma, beta, mean, rstd, relu, (const bf16*)skip, lds_, relu_sum, (bf16*)y, ldy, s, ch);
  };
  if (ldy == NARROW_PITCH) launch(std::integral_constant<int, 4>());
  else launch(std::integral_constant<int, 8>());
  return ok("bn_forward");
}

int launch_bn_backward(const void* dy, int64_t ldd, const void* x, int64_t ldx, int C,
                       const float* gamma, const float* mean, const float* rstd, float* scratch,
                       float* dgamma, float* dbeta, int64_t group_stride, int need_dx,
                       int relu_below, void* dx, int64_t ldo, const Segs& s, void* stream) {
  const int rows = s.off[s.K];
  if (C == 0) return DYNB_OK;
  const Chunks ch = make_chunks(s);
  const int nch = ch.first[s.K];
  float* pdg = scratch;
  float* pdb = scratch + (int64_t)nch * C;
  // algorithmic bytes: dy and x read once, dx written once (the kernels read dy and x twice)
  Timed t(KC_NORM, stream, 0, (double)rows * C * (need_dx ? 6 : 4));
  const hipStream_t st = (hipStream_t)stream;
  auto launch = [&](auto lpr) {
    constexpr int LPR = decltype(lpr)::value, COLS = 8 * LPR;
    if (nch > 0)
      hipLaunchKernelGGL(bn_chunk_param_grad_kernel<LPR>, dim3(nch, (C + COLS - 1) / COLS), dim3(32 * LPR), 0, st,
                         (const bf16*)dy, ldd, (const bf16*)x, ldx, C, mean, rstd, pdg, pdb, s, ch);
    hipLaunchKernelGGL(bn_merge_param_grad_kernel, dim3((C + MERGE_C - 1) / MERGE_C, s.K), dim3(1024), 0, st, pdg,
                       pdb, C, dgamma, dbeta, group_stride, ch);
    if (need_dx && nch > 0)   // (padding columns that no block covers hold zeros and keep them)
      hipLaunchKernelGGL(bn_input_grad_kernel<LPR>, dim3(nch, (C + COLS - 1) / COLS), dim3(32 * LPR), 0, st,
                         (const bf16*)dy, ldd, (const bf16*)x, ldx, C, gamma, mean, rstd, dgamma, dbeta,
                         group_stride, relu_below, (bf16*)dx, ldo, s, ch);
  };
  if (ldd == NARROW_PITCH) launch(std::integral_constant<int, 4>());
  else launch(std::integral_constant<int, 8>());
  return ok("bn_backward");
}

int64_t row_scratch_floats(int64_t max_rows, int max_workers, int C) {
  return 2 * ((max_rows + CHUNK_ROWS - 1) / CHUNK_ROWS + max_workers) * (int64_t)C;
}

int launch_add_forward(const void* a, int64_t lda, const void* b, int64_t ldb, int64_t width,
                       int64_t rows, int relu, void* out, int64_t ldo, void* stream) {
  if (rows == 0 || width == 0) return DYNB_OK;
  const int gpr = (int)(width / 8);
  const int64_t total = rows * gpr;
  Timed t(KC_NORM, stream, 0, (double)rows * width * 6);
  hipLaunchKernelGGL(add_forward_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0,
                     (hipStream_t)stream, (const bf16*)a, lda, (const bf16*)b, ldb, gpr, total, relu,
                     (bf16*)out, ldo);
  return ok("add_forward");
}

int launch_grad_route(const void* src, int64_t lds_, const void* act, int64_t lda, int64_t width,
                      int64_t rows, int relu, int accumulate, void* dst, int64_t ldd, void* stream) {
  if (rows == 0 || width == 0) return DYNB_OK;
  const int gpr = (int)(width / 8);
  const int64_t total = rows * gpr;
  Timed t(KC_NORM, stream, 0, (double)rows * width * (2 + 2 + (relu ? 2 : 0) + (accumulate ? 2 : 0)));
  hipLaunchKernelGGL(grad_route_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0,
                     (hipStream_t)stream, (const bf16*)src, lds_, (const bf16*)act, lda, gpr, total,
                     relu, accumulate, (bf16*)dst, ldd);
  return ok("grad_route");
}

}  // namespace dynb
