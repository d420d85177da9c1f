// Optimizer steps on the flat fp32 parameter vector: plain SGD (Eq. 3), heavy-ball momentum and
// Adam (the optimizers of the paper's workloads), optionally with the weighted aggregation of
// Eq. 2 folded in (the K per-worker gradients are read and summed where the step is applied, so
// the aggregate never goes through HBM), and fused with the refresh of the 16-bit weight copies.
#include <hip/hip_runtime.h>

#include <cmath>

#include "dynb_internal.h"

namespace dynb {
namespace {

typedef __bf16 bf16;
typedef float f4 __attribute__((ext_vector_type(4)));

template <typename T> __device__ inline T from_float(float v) { return (T)v; }

// One parameter, one step.  s1/s2 are the optimizer's state for this parameter.
constexpr int COPY_ONLY = -1;   // no step: only the copies of the weights as they are
template <int KIND>
__device__ inline float step_one(const UpdateRule& r, float w, float g, float& s1, float& s2) {
  if (KIND == COPY_ONLY) return w;
  if (KIND == DYNB_OPT_SGD) return w - r.lr * g;
  if (KIND == DYNB_OPT_MOMENTUM) {
    s1 = r.mu * s1 + g;
    return w - r.lr * s1;
  }
  s1 = r.beta1 * s1 + r.omb1 * g;
  s2 = r.beta2 * s2 + r.omb2 * g * g;
  return w - r.lr * (s1 * r.inv_c1) / (sqrtf(s2 * r.inv_c2) + r.eps);
}

// Gradient of 4 consecutive parameters starting at o (16-byte aligned).
template <bool AGG>
__device__ inline f4 gradient4(const GradSource& src, int64_t o) {
  if (!AGG) return *(const f4*)(src.g + o);
  constexpr int U = 8;   // loads in flight per lane
  f4 acc = {0.f, 0.f, 0.f, 0.f};
  int k = 0;
  for (; k + U <= src.lam.K; k += U) {
    f4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      v[u] = __builtin_nontemporal_load((const f4*)(src.g + (int64_t)(k + u) * src.worker_stride + o));
#pragma unroll
    for (int u = 0; u < U; ++u) acc += src.lam.w[k + u] * v[u];
  }
  for (; k < src.lam.K; ++k)
    acc += src.lam.w[k] *
           __builtin_nontemporal_load((const f4*)(src.g + (int64_t)k * src.worker_stride + o));
  return acc;
}
template <bool AGG>
__device__ inline float gradient1(const GradSource& src, int64_t o) {
  if (!AGG) return src.g[o];
  float acc = 0.f;
  for (int k = 0; k < src.lam.K; ++k) acc += src.lam.w[k] * src.g[(int64_t)k * src.worker_stride + o];
  return acc;
}

// Gradients of U parameters at o[0..U): every load of a worker's U elements, and of four workers, is
// in flight at once (ascending k per element, as above).
template <bool AGG, int U>
__device__ inline void gradients(const GradSource& src, const int64_t (&o)[U], float (&g)[U]) {
  if (!AGG) {
#pragma unroll
    for (int u = 0; u < U; ++u) g[u] = src.g[o[u]];
    return;
  }
#pragma unroll
  for (int u = 0; u < U; ++u) g[u] = 0.f;
  const float* base = src.g;
  int k = 0;
  for (; k + 4 <= src.lam.K; k += 4, base += 4 * src.worker_stride) {
    float v[4][U];
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
      for (int u = 0; u < U; ++u) v[w][u] = base[w * src.worker_stride + o[u]];
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
      for (int u = 0; u < U; ++u) g[u] += src.lam.w[k + w] * v[w][u];
  }
  for (; k < src.lam.K; ++k, base += src.worker_stride)
#pragma unroll
    for (int u = 0; u < U; ++u) g[u] += src.lam.w[k] * base[o[u]];
}

// ---- weight matrices: step + both 16-bit copies in one pass ----------------------------------
// W[r][c] <- step(W[r][c]); Wn[r][c] = T(W), Wt[c][r] = T(W).  (A convolution is nine such matrices,
// one per tap, whose copies lie side by side in the rows of its two operands.)  A workgroup owns a TR x TC tile:
// 16-byte accesses on the fp32 side, the transposed copy goes through an LDS tile so that its
// stores are 16 bytes per lane and whole 128-byte lines per 8 (bf16) lanes.
// One launch serves every matrix of `mats` (workgroups mats.first_block[i] ... belong to matrix
// i) and, with the workgroups behind the last tile, the small tensors of `small` (biases):
// back-to-back launches on one stream leave the chip idle for a few microseconds each, which
// for a four-layer model came to a sixth of the whole update.
template <typename T, int KIND, bool AGG, int TC, int TR>
__device__ __forceinline__ void update_tile(int blk, float* __restrict__ params, const CastMats& mats,
                                            const GradSource& src, const UpdateRule& rule,
                                            float* __restrict__ s1, float* __restrict__ s2) {
  constexpr bool HAS_S1 = KIND == DYNB_OPT_MOMENTUM || KIND == DYNB_OPT_ADAM;
  int mi = 0;
  while (blk >= mats.first_block[mi + 1]) ++mi;
  const int64_t ldn = mats.ldn[mi], ldt = mats.ldt[mi];
  const int R = mats.R[mi], C = mats.C[mi];
  const int tiles_x = (C + TC - 1) / TC, local = blk - mats.first_block[mi];
  const int per_tap = tiles_x * ((R + TR - 1) / TR), tap = local / per_tap, in_tap = local - tap * per_tap;
  const int tile_x = in_tap % tiles_x, tile_y = in_tap / tiles_x;
  const int64_t off = mats.off[mi] + (int64_t)tap * R * C;
  T* __restrict__ Wn = (T*)mats.Wn[mi] + tap * mats.tap_n[mi];
  T* __restrict__ Wt = (T*)mats.Wt[mi] + tap * mats.tap_t[mi];
  constexpr int G = 16 / sizeof(T);
  typedef T vecT __attribute__((ext_vector_type(G)));
  typedef T vec4T __attribute__((ext_vector_type(4)));
  constexpr int QC = TC / 4;   // 16-byte granules per tile row
  __shared__ float tile[TR][TC + 1];
  const int r0 = tile_y * TR, c0 = tile_x * TC;
  // 16-byte accesses need aligned rows in every array (all start at a multiple of 4 floats);
  // otherwise a lane takes single elements, U of the tile's elements row after row, 256 apart, at once.
  // (1001 x 2050 and 2050 x 777, 7 workers, Adam: 106 us with four elements in turn
  // per lane -> 43 us, what its 210 MB take at the rate of a large copy.)
  const bool vec = (C & 3) == 0 && (off & 3) == 0;
  if (!vec) {
    // (only the elements that exist: rows of a head of ten classes are one round, not several; more in flight
    // would cost the aligned path its occupancy)
    constexpr int U = 4;
    const int cols = min(TC, C - c0), total = cols * min(TR, R - r0);
    for (int idx = threadIdx.x; idx < total; idx += 256 * U) {
      int64_t o[U];
      int er[U], ec[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = idx + 256 * u < total ? idx + 256 * u : idx;   // (a dead lane repeats its first)
        er[u] = e / cols;
        ec[u] = e - er[u] * cols;
        o[u] = off + (int64_t)(r0 + er[u]) * C + c0 + ec[u];
      }
      float g[U], w[U], a[U], b[U];
      if (KIND != COPY_ONLY) gradients<AGG, U>(src, o, g);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        w[u] = params[o[u]];
        a[u] = HAS_S1 ? s1[o[u]] : 0.f;
        b[u] = KIND == DYNB_OPT_ADAM ? s2[o[u]] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        w[u] = step_one<KIND>(rule, w[u], g[u], a[u], b[u]);
        if (idx + 256 * u >= total) continue;
        if (KIND != COPY_ONLY) params[o[u]] = w[u];
        if (HAS_S1) s1[o[u]] = a[u];
        if (KIND == DYNB_OPT_ADAM) s2[o[u]] = b[u];
        Wn[(int64_t)(r0 + er[u]) * ldn + c0 + ec[u]] = from_float<T>(w[u]);
        tile[er[u]][ec[u]] = w[u];
      }
    }
  } else {
#pragma unroll 2
    for (int idx = threadIdx.x; idx < TR * QC; idx += 256) {
      const int r = idx / QC, cq = (idx % QC) * 4;
      const int gr = r0 + r, gc = c0 + cq;
      f4 w = {0.f, 0.f, 0.f, 0.f};
      if (gr < R && gc < C) {
        const int64_t o = off + (int64_t)gr * C + gc;
        f4 a = {0.f, 0.f, 0.f, 0.f}, b = a, d = a;
        if (KIND != COPY_ONLY) d = gradient4<AGG>(src, o);
        w = *(const f4*)(params + o);
        if (HAS_S1) a = *(const f4*)(s1 + o);
        if (KIND == DYNB_OPT_ADAM) b = *(const f4*)(s2 + o);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float ae = a[e], be = b[e];
          w[e] = step_one<KIND>(rule, w[e], d[e], ae, be);
          a[e] = ae;
          b[e] = be;
        }
        if (KIND != COPY_ONLY) *(f4*)(params + o) = w;
        if (HAS_S1) *(f4*)(s1 + o) = a;
        if (KIND == DYNB_OPT_ADAM) *(f4*)(s2 + o) = b;
        const vec4T q = {from_float<T>(w[0]), from_float<T>(w[1]), from_float<T>(w[2]), from_float<T>(w[3])};
        *(vec4T*)(Wn + (int64_t)gr * ldn + gc) = q;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) tile[r][cq + e] = w[e];
    }
  }
  __syncthreads();
  constexpr int GR = TR / G;   // granules of rows per tile column
  for (int idx = threadIdx.x; idx < TC * GR; idx += 256) {
    const int rg = idx % GR, c = idx / GR;
    if (c0 + c >= C) continue;
    if (r0 + rg * G + G <= R) {
      vecT v;
#pragma unroll
      for (int e = 0; e < G; ++e) v[e] = from_float<T>(tile[rg * G + e][c]);
      *(vecT*)(Wt + (int64_t)(c0 + c) * ldt + r0 + rg * G) = v;
    } else {
      for (int e = 0; e < G && r0 + rg * G + e < R; ++e)
        Wt[(int64_t)(c0 + c) * ldt + r0 + rg * G + e] = from_float<T>(tile[rg * G + e][c]);
    }
  }
}

template <typename T, int KIND, bool AGG, int TC, int TR>
__global__ __launch_bounds__(256) void update_cast_kernel(float* __restrict__ params, CastMats mats,
                                                          Ranges small, int range_blocks,
                                                          GradSource src, UpdateRule rule,
                                                          float* __restrict__ s1,
                                                          float* __restrict__ s2) {
  constexpr bool HAS_S1 = KIND == DYNB_OPT_MOMENTUM || KIND == DYNB_OPT_ADAM;
  const int blk = blockIdx.x;
  if (blk >= mats.first_block[mats.n]) {   // the small tensors, element by element
    const int rb = blk - mats.first_block[mats.n];
    for (int q = 0; q < small.n; ++q) {
      const int64_t off = small.off[q], n = small.len[q];
      for (int64_t i = (int64_t)rb * 256 + threadIdx.x; i < n; i += (int64_t)range_blocks * 256) {
        const int64_t o = off + i;
        float a = HAS_S1 ? s1[o] : 0.f;
        float b = KIND == DYNB_OPT_ADAM ? s2[o] : 0.f;
        params[o] = step_one<KIND>(rule, params[o], gradient1<AGG>(src, o), a, b);
        if (HAS_S1) s1[o] = a;
        if (KIND == DYNB_OPT_ADAM) s2[o] = b;
      }
    }
    return;
  }
  update_tile<T, KIND, AGG, TC, TR>(blk, params, mats, src, rule, s1, s2);
}

// ---- everything a dense model's scratch needs before a pass over it, in one launch ---------------
// The weight copies, the packed input (padding columns included) and zeros in the padding columns of what
// later kernels write only in part: workgroups of each kind behind those of the one before.  What bounds it is one
// workgroup's chain, so every tensor to be padded has workgroups of its own (all tensors in turn in each: 10-7-5-8-17,
// four workers, whole call 37.5 -> 28.8 us).
template <typename T, int TR>
__global__ __launch_bounds__(256) void prepare_kernel(const float* __restrict__ params, CastMats mats, Prepare pr,
                                                      int pack_blocks, int pad_blocks) {
  int blk = blockIdx.x;
  if (blk < mats.first_block[mats.n]) {
    const GradSource src = {};
    const UpdateRule rule = {};
    update_tile<T, COPY_ONLY, false, 64, TR>(blk, const_cast<float*>(params), mats, src, rule, nullptr, nullptr);
    return;
  }
  blk -= mats.first_block[mats.n];
  if (blk < pack_blocks) {                 // eight columns of a row per lane
    typedef T vec8T __attribute__((ext_vector_type(8)));
    const uint32_t gpr = (uint32_t)(pr.ld / 8), total = (uint32_t)pr.rows * gpr;
    for (uint32_t i = (uint32_t)blk * 256 + threadIdx.x; i < total; i += (uint32_t)pack_blocks * 256) {
      const int64_t r = i / gpr;
      const int c = (int)(i % gpr) * 8;
      vec8T v;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float t = pr.x[r * pr.D + (c + e < pr.D ? c + e : 0)];
        v[e] = c + e < pr.D ? from_float<T>(t) : from_float<T>(0.f);
      }
      *(vec8T*)((T*)pr.act + r * pr.ld + c) = v;
    }
    return;
  }
  blk -= pack_blocks;                      // pad_blocks for each tensor
  const int q = blk / pad_blocks, ld = pr.pad_ld[q];
  const uint32_t w = (uint32_t)(ld - pr.pad_from[q]), total = (uint32_t)pr.pad_rows[q] * w;
  T* const p = (T*)pr.pad[q] + pr.pad_from[q];
  for (uint32_t i = (uint32_t)(blk - q * pad_blocks) * 256 + threadIdx.x; i < total; i += (uint32_t)pad_blocks * 256)
    p[(int64_t)(i / w) * ld + i % w] = from_float<T>(0.f);
}

// ---- element-wise step over a list of ranges (blockIdx.y = range) ---------------------------
template <int KIND, bool AGG>
__global__ __launch_bounds__(256) void update_ranges_kernel(float* __restrict__ params, Ranges r,
                                                            GradSource src, UpdateRule rule,
                                                            float* __restrict__ s1,
                                                            float* __restrict__ s2) {
  const int64_t off = r.off[blockIdx.y], n = r.len[blockIdx.y];
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int64_t o = off + i;
    float a = KIND != DYNB_OPT_SGD ? s1[o] : 0.f;
    float b = KIND == DYNB_OPT_ADAM ? s2[o] : 0.f;
    params[o] = step_one<KIND>(rule, params[o], gradient1<AGG>(src, o), a, b);
    if (KIND != DYNB_OPT_SGD) s1[o] = a;
    if (KIND == DYNB_OPT_ADAM) s2[o] = b;
  }
}

// ---- plain streaming Adam ----------------------------------------------------------------------
__global__ __launch_bounds__(256) void adam_kernel(f4* __restrict__ x, f4* __restrict__ m,
                                                   f4* __restrict__ v, const f4* __restrict__ g,
                                                   int64_t n4, UpdateRule rule) {
  const int64_t stride = (int64_t)gridDim.x * 256;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += stride) {
    f4 p = x[i], a = m[i], b = v[i];
    const f4 d = g[i];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float ae = a[e], be = b[e];
      p[e] = step_one<DYNB_OPT_ADAM>(rule, p[e], d[e], ae, be);
      a[e] = ae;
      b[e] = be;
    }
    x[i] = p;
    m[i] = a;
    v[i] = b;
  }
}

inline int ok(const char* what) {
  return hipGetLastError() == hipSuccess ? DYNB_OK : fail(DYNB_ERR_HIP, "%s: launch failed", what);
}

// algorithmic bytes per parameter of one step: parameter read + write, each state read + write,
// and the gradient (one read, or K reads when aggregating on the fly)
double bytes_per_param(const UpdateRule& rule, const GradSource& src) {
  const int states = rule.kind == DYNB_OPT_ADAM ? 2 : rule.kind == DYNB_OPT_MOMENTUM ? 1 : 0;
  return 8.0 + 8.0 * states + 4.0 * (src.lam.K > 0 ? src.lam.K : 1);
}
double flops_per_param(const UpdateRule& rule, const GradSource& src) {
  const double step = rule.kind == DYNB_OPT_ADAM ? 14.0 : rule.kind == DYNB_OPT_MOMENTUM ? 4.0 : 2.0;
  return step + (src.lam.K > 0 ? 2.0 * src.lam.K : 0.0);
}

// (wider tiles when K gradient streams are read: 512-byte runs per row and stream)
constexpr int cast_tile_columns(bool agg) { return agg ? 128 : 64; }
constexpr int SHORT_ROWS = 16, TALL_ROWS = 64;

template <typename T, int KIND, bool AGG>
void launch_update_cast_t(float* params, const CastMats& mats, int rows, const Ranges& small, int range_blocks,
                          const GradSource& src, const UpdateRule& rule, float* s1, float* s2,
                          hipStream_t st) {
  constexpr int TC = cast_tile_columns(AGG);
  const dim3 grid((unsigned)(mats.first_block[mats.n] + range_blocks));
  if (rows == SHORT_ROWS)
    hipLaunchKernelGGL((update_cast_kernel<T, KIND, AGG, TC, SHORT_ROWS>), grid, dim3(256), 0, st, params, mats,
                       small, range_blocks, src, rule, s1, s2);
  else
    hipLaunchKernelGGL((update_cast_kernel<T, KIND, AGG, TC, TALL_ROWS>), grid, dim3(256), 0, st, params, mats,
                       small, range_blocks, src, rule, s1, s2);
}

template <typename T, int KIND>
void launch_update_cast_k(float* params, const CastMats& mats, int rows, const Ranges& small, int range_blocks,
                          const GradSource& src, const UpdateRule& rule, float* s1, float* s2,
                          hipStream_t st) {
  if (src.lam.K > 0)
    launch_update_cast_t<T, KIND, true>(params, mats, rows, small, range_blocks, src, rule, s1, s2, st);
  else
    launch_update_cast_t<T, KIND, false>(params, mats, rows, small, range_blocks, src, rule, s1, s2, st);
}

template <typename T>
void launch_update_cast_d(float* params, const CastMats& mats, int rows, const Ranges& small, int range_blocks,
                          const GradSource& src, const UpdateRule& rule, float* s1, float* s2,
                          hipStream_t st) {
  switch (rule.kind) {
    case DYNB_OPT_SGD:
      launch_update_cast_k<T, DYNB_OPT_SGD>(params, mats, rows, small, range_blocks, src, rule, s1, s2, st);
      break;
    case DYNB_OPT_MOMENTUM:
      launch_update_cast_k<T, DYNB_OPT_MOMENTUM>(params, mats, rows, small, range_blocks, src, rule, s1, s2, st);
      break;
    default:
      launch_update_cast_k<T, DYNB_OPT_ADAM>(params, mats, rows, small, range_blocks, src, rule, s1, s2, st);
  }
}

// Fills first_block and counts the parameters of `mats`.
int count_blocks(CastMats& mats, int tile_columns, int tile_rows, double& params_counted) {
  if (mats.n < 0 || mats.n > MAX_CAST_MATS) return fail(DYNB_ERR_BADARG, "update_cast: too many tensors for one launch");
  int64_t blocks = 0;
  params_counted = 0.0;
  for (int i = 0; i < mats.n; ++i) {
    if (mats.R[i] <= 0 || mats.C[i] <= 0) return fail(DYNB_ERR_BADARG, "update_cast: empty matrix");
    mats.first_block[i] = (int)blocks;
    blocks += (int64_t)((mats.C[i] + tile_columns - 1) / tile_columns) * ((mats.R[i] + tile_rows - 1) / tile_rows) * mats.taps[i];
    if (blocks >= ((int64_t)1 << 31) - 256)
      return fail(DYNB_ERR_UNSUPPORTED, "update_cast: too many tiles for one launch");
    params_counted += (double)mats.R[i] * mats.C[i] * mats.taps[i];
  }
  for (int i = mats.n; i <= MAX_CAST_MATS; ++i) mats.first_block[i] = (int)blocks;
  return DYNB_OK;
}

}  // namespace

// A tile of 64 rows is a chain of four to sixteen rounds of loads and stores in one workgroup; with fewer tiles than
// compute units that chain is the launch, and tiles of 16 rows shorten it: Adam on 785-301-97-10, 79 -> 297 workgroups,
// 10.6 -> 6.5 us; 32-64-128 convolutions, 39 -> 108, 5.3 -> 4.6.  From there on it is the bytes (3072-512-512-10: 458
// workgroups 8.1, 1826 8.0), and tall tiles write the transposed copy in whole lines.
// With the average of K workers folded in, a workgroup walks K gradients, and four times as many of them cost more
// than shorter chains save once K, the matrices and the tiles or bytes are not few.  Time of the launch, between the
// others of an iteration, on short tiles over tall ones, dense models (2000, 2 to 64 workers): below 8 workers 0.58 (1.02 at
// most); one or two layers 0.60 to 0.77, at any size; from three layers and 8 workers on, below 64 tiles 0.6 to 0.98, 128 to
// 256 1.0 to 1.4 from 16 workers on; more than 100 MB of gradients 1.06 to 1.3; six layers or more 0.95 to 1.05 (the
// biases of every layer are chains of their own beside the tiles).  Convolutions (568 models): below 40 MB 0.78, 40 to 64
// MB 1.07, above 1.2 (320-320 channels, 32 workers, 30 -> 41 us).
int cast_tile_rows(const CastMats& mats, int tile_columns, int K) {
  int64_t tall = 0, weights = 0;
  bool conv = false;
  for (int i = 0; i < mats.n && i < MAX_CAST_MATS; ++i) {
    tall += (int64_t)((mats.C[i] + tile_columns - 1) / tile_columns) * ((mats.R[i] + TALL_ROWS - 1) / TALL_ROWS) * mats.taps[i];
    weights += (int64_t)mats.taps[i] * mats.R[i] * mats.C[i];
    conv = conv || mats.taps[i] > 1;
  }
  const bool few = K < 8 || (mats.n <= 2 && !conv) ||
                   (tall < 128 && 4 * K * weights < 48000000 && mats.n <= (K < 16 ? 6 : 5));
  return tall < 256 && few ? SHORT_ROWS : TALL_ROWS;
}

int launch_update_cast(int dtype, float* params, CastMats& mats, const Ranges& small,
                       const GradSource& src, const UpdateRule& rule, float* s1, float* s2,
                       void* stream) {
  if (small.n < 0 || small.n > MAX_RANGES)
    return fail(DYNB_ERR_BADARG, "update_cast: too many tensors for one launch");
  const int es = dtype == DYNB_BF16 ? 2 : 4;
  double cast_n = 0.0, small_n = 0.0;
  int64_t longest = 0;
  const int columns = cast_tile_columns(src.lam.K > 0), rows = cast_tile_rows(mats, columns, src.lam.K);
  if (int rc = count_blocks(mats, columns, rows, cast_n)) return rc;
  for (int i = 0; i < small.n; ++i) {
    longest = small.len[i] > longest ? small.len[i] : longest;
    small_n += (double)small.len[i];
  }
  int64_t range_blocks = (longest + 255) / 256;
  if (range_blocks > 256) range_blocks = 256;
  if (mats.first_block[mats.n] + range_blocks == 0) return DYNB_OK;
  Timed t(KC_UPDATE, stream, flops_per_param(rule, src) * (cast_n + small_n),
          (bytes_per_param(rule, src) + 2 * es) * cast_n + bytes_per_param(rule, src) * small_n);
  if (dtype == DYNB_BF16)
    launch_update_cast_d<bf16>(params, mats, rows, small, (int)range_blocks, src, rule, s1, s2, (hipStream_t)stream);
  else
    launch_update_cast_d<float>(params, mats, rows, small, (int)range_blocks, src, rule, s1, s2, (hipStream_t)stream);
  return ok("update_cast");
}

int launch_weight_casts(int dtype, const float* params, CastMats& mats, void* stream) {
  const int es = dtype == DYNB_BF16 ? 2 : 4;
  double n = 0.0;
  const int rows = cast_tile_rows(mats, cast_tile_columns(false), 0);
  if (int rc = count_blocks(mats, cast_tile_columns(false), rows, n)) return rc;
  if (n == 0.0) return DYNB_OK;
  Timed t(KC_WEIGHT_CAST, stream, 0, n * (4 + 2 * es));
  Ranges none;
  none.n = 0;
  const GradSource src = {};
  const UpdateRule rule = {};
  if (dtype == DYNB_BF16)
    launch_update_cast_t<bf16, COPY_ONLY, false>(const_cast<float*>(params), mats, rows, none, 0, src, rule,
                                                 nullptr, nullptr, (hipStream_t)stream);
  else
    launch_update_cast_t<float, COPY_ONLY, false>(const_cast<float*>(params), mats, rows, none, 0, src, rule,
                                                  nullptr, nullptr, (hipStream_t)stream);
  return ok("weight_casts");
}

int launch_prepare(int dtype, const float* params, CastMats& mats, const Prepare& pr, void* stream) {
  const int es = dtype == DYNB_BF16 ? 2 : 4;
  double n = 0.0;
  const int rows = cast_tile_rows(mats, cast_tile_columns(false), 0);
  if (int rc = count_blocks(mats, cast_tile_columns(false), rows, n)) return rc;
  const int64_t granules = (int64_t)pr.rows * (pr.ld / 8);
  int64_t pads = 0;
  for (int q = 0; q < pr.n; ++q) {
    const int64_t t = (int64_t)pr.pad_rows[q] * (pr.pad_ld[q] - pr.pad_from[q]);
    pads = t > pads ? t : pads;
  }
  const int pack_blocks = (int)(granules / 256 < 2048 ? (granules + 255) / 256 : 2048);
  // (32-bit indices, with room for a grid's step behind the last: the scratch of a call is far below)
  if (granules >= (int64_t)1 << 30 || pads >= (int64_t)1 << 30)
    return fail(DYNB_ERR_UNSUPPORTED, "prepare: tensors too large for 32-bit indices");
  const int64_t most = pr.n > 0 ? 1024 / pr.n : 1;
  const int pad_blocks = (int)((pads + 1023) / 1024 < most ? (pads + 1023) / 1024 : most);
  const int blocks = mats.first_block[mats.n] + pack_blocks + pr.n * pad_blocks;
  if (blocks == 0) return DYNB_OK;
  Timed t(KC_WEIGHT_CAST, stream, 0, n * (4 + 2 * es) + (double)pr.rows * pr.D * (4 + es));
  const auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(256), 0, (hipStream_t)stream, params, mats, pr, pack_blocks, pad_blocks);
  };
  if (dtype == DYNB_BF16)
    launch(rows == SHORT_ROWS ? prepare_kernel<bf16, SHORT_ROWS> : prepare_kernel<bf16, TALL_ROWS>);
  else
    launch(rows == SHORT_ROWS ? prepare_kernel<float, SHORT_ROWS> : prepare_kernel<float, TALL_ROWS>);
  return ok("prepare");
}

void set_adam(UpdateRule& r, double beta1, double beta2, float eps, int64_t t) {
  r.beta1 = (float)beta1;
  r.beta2 = (float)beta2;
  r.omb1 = (float)(1.0 - beta1);
  r.omb2 = (float)(1.0 - beta2);
  r.eps = eps;
  r.inv_c1 = (float)(1.0 / (1.0 - std::pow(beta1, (double)t)));
  r.inv_c2 = (float)(1.0 / (1.0 - std::pow(beta2, (double)t)));
}

namespace {
template <int KIND>
void launch_update_ranges_k(float* params, const Ranges& r, const GradSource& src, const UpdateRule& rule,
                            float* s1, float* s2, dim3 grid, hipStream_t st) {
  if (src.lam.K > 0)
    hipLaunchKernelGGL((update_ranges_kernel<KIND, true>), grid, dim3(256), 0, st, params, r, src, rule, s1, s2);
  else
    hipLaunchKernelGGL((update_ranges_kernel<KIND, false>), grid, dim3(256), 0, st, params, r, src, rule, s1, s2);
}
}  // namespace

int launch_update_ranges(float* params, const Ranges& r, const GradSource& src, const UpdateRule& rule,
                         float* s1, float* s2, void* stream) {
  int64_t longest = 0, total = 0;
  for (int i = 0; i < r.n; ++i) {
    longest = r.len[i] > longest ? r.len[i] : longest;
    total += r.len[i];
  }
  if (r.n <= 0 || longest <= 0) return DYNB_OK;
  Timed t(KC_UPDATE, stream, flops_per_param(rule, src) * total, bytes_per_param(rule, src) * total);
  int64_t bx = (longest + 255) / 256;
  if (bx > 1024) bx = 1024;
  const dim3 grid((unsigned)bx, r.n);
  switch (rule.kind) {
    case DYNB_OPT_SGD:
      launch_update_ranges_k<DYNB_OPT_SGD>(params, r, src, rule, s1, s2, grid, (hipStream_t)stream);
      break;
    case DYNB_OPT_MOMENTUM:
      launch_update_ranges_k<DYNB_OPT_MOMENTUM>(params, r, src, rule, s1, s2, grid, (hipStream_t)stream);
      break;
    default:
      launch_update_ranges_k<DYNB_OPT_ADAM>(params, r, src, rule, s1, s2, grid, (hipStream_t)stream);
  }
  return ok("update_ranges");
}

int launch_adam(float* params, float* m, float* v, const float* g, int64_t n,
                const UpdateRule& rule, void* stream) {
  const int64_t n4 = n / 4;
  if (n4 == 0) return DYNB_OK;
  Timed t(KC_UPDATE, stream, 14.0 * n, 28.0 * n);
  int64_t bx = (n4 + 255) / 256;
  if (bx > 256 * 16) bx = 256 * 16;
  hipLaunchKernelGGL(adam_kernel, dim3((unsigned)bx), dim3(256), 0, (hipStream_t)stream, (f4*)params,
                     (f4*)m, (f4*)v, (const f4*)g, n4, rule);
  return ok("adam");
}

}  // namespace dynb

using namespace dynb;

extern "C" int dynb_adam_update(float* params, float* m, float* v, const float* g, int64_t n,
                                float lr, double beta1, double beta2, float eps, int64_t step,
                                void* stream) {
  if (!params || !m || !v || !g) return fail(DYNB_ERR_BADARG, "adam: null pointer");
  if (n < 0 || (n & 3)) return fail(DYNB_ERR_BADARG, "adam: n must be a non-negative multiple of 4");
  if (((uintptr_t)params | (uintptr_t)m | (uintptr_t)v | (uintptr_t)g) & 15)
    return fail(DYNB_ERR_BADARG, "adam: pointers must be 16-byte aligned");
  if (step < 1) return fail(DYNB_ERR_BADARG, "adam: step numbers start at 1");
  if (!(beta1 >= 0.0 && beta1 < 1.0 && beta2 >= 0.0 && beta2 < 1.0))
    return fail(DYNB_ERR_BADARG, "adam: betas must lie in [0, 1)");
  UpdateRule r{};
  r.kind = DYNB_OPT_ADAM;
  r.lr = lr;
  set_adam(r, beta1, beta2, eps, step);
  return launch_adam(params, m, v, g, n, r, stream);
}
