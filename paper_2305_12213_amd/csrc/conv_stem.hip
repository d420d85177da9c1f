// The first convolution of a model (3x3, zero padding 1, stride 1 or 2) on images of at most three
// channels: forward and weight gradient straight from the caller's fp32 pixels (rounded to bf16
// where they are read, as a packed copy would be).  Its reduction is 9 x 3 = 27 long, less than two
// matrix-instruction steps, so it is bound by the one wide tensor next to it -- the output, or the
// gradient wrt it.  The general kernels pad the input to 64 channels (a packed copy of which 16 of 128
// bytes are used, and 64 x 64 products of which 3 x 64 count).
// 512 x 32 x 32 x 3 -> 64 channels, per iteration: packing 17 us, forward 57, weight gradient 54 + 7
// -> forward 24, weight gradient 24 + 5 (the 67 MB of the wide tensor take 10 us to write, 14 to read).
#include <hip/hip_runtime.h>

#include "device_rows.h"
#include "dynb_internal.h"
#include "lds_async.h"

namespace dynb {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

struct StemArgs {
  const float* x; int H, W;          // [images * H * W][CIN]
  int Ho, Wo, stride;
  int64_t pixels;                    // output pixels: images * Ho * Wo
  // forward
  const bf16* w; int kf;             // [N][kf]: w[co][tap * 8 + ci], kf >= 80
  const float* bias; int N, relu;
  bf16* out; int64_t ldo;            // [pixels][ldo], whole 32-channel blocks
  // weight gradient
  const bf16* dy; int64_t ldd;       // [pixels][ldd]
  float* partial;                    // [chunk][64-channel block][PART] chunk results
  const void* zeros;
};

// The CIN channels under tap `tap` of output pixel (image img, oy, ox); zeros outside the image or
// where !live.
template <int CIN>
__device__ inline void fetch_tap(const StemArgs& p, int img, int oy, int ox, int tap, bool live, float (&v)[CIN]) {
  const int sy = oy * p.stride + tap / 3 - 1, sx = ox * p.stride + tap % 3 - 1;
  const bool ok = live && sy >= 0 && sy < p.H && sx >= 0 && sx < p.W;
  const float* src = p.x + (ok ? ((int64_t)(img * p.H + sy) * p.W + sx) * CIN : 0);
#pragma unroll
  for (int c = 0; c < CIN; ++c) {
    const float t = src[c];          // (pixel 0 where nothing is to be read: the batch is not empty)
    v[c] = ok ? t : 0.f;
  }
}

// A workgroup takes 256 output pixels x 64 output channels, a wave 64 pixels.  A matrix-instruction step is two
// taps x 8 channels, as the weight copies lie in memory (their padding and the tenth tap are zeros; five steps,
// in the order of the general kernel), one tap per lane half: a lane gathers its operand's channels of its own two
// pixels straight into registers.  The results pass through LDS, 32 pixels at a time, so that a store writes
// whole rows; padding channels are written as zeros.  Up to 32 channels the upper half is left out.
// What bounds a launch is the latency of these gathers, so little LDS and many waves: 512 x 32 x 32 x 3 -> 64
// 24 us (with the patches of all nine taps built in LDS, two workgroups per compute unit: 27), -> 32 18 (23).
constexpr int WPITCH = 176, OPITCH = 144;  // bytes per weight row, result (odd multiples of 16: no bank conflicts)

template <int CIN>
__global__ __launch_bounds__(256) void stem_forward_kernel(StemArgs p) {
  __shared__ __align__(16) char area[4][32 * OPITCH];
  __shared__ __align__(16) char wl[64 * WPITCH];
  __shared__ __align__(16) float bl[64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l31 = lane & 31, h = lane >> 5;
  const int j0 = blockIdx.y * 64;
  const bool upper = p.N - j0 > 32;
  const int64_t pix0 = (int64_t)blockIdx.x * 256 + wave * 64;
  float v[2][5][CIN];                                      // [pixel][step]: tap 2 step + h
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const int64_t pix = pix0 + a * 32 + l31;
    const bool live = pix < p.pixels;
    const int q = live ? (int)pix : 0, row = q / p.Wo, ox = q - row * p.Wo, img = row / p.Ho, oy = row - img * p.Ho;
#pragma unroll
    for (int kk = 0; kk < 5; ++kk) fetch_tap<CIN>(p, img, oy, ox, 2 * kk + h, live && 2 * kk + h < 9, v[a][kk]);
  }
  for (int e = threadIdx.x; e < 64 * 10; e += 256) {       // weights: ten granules per channel
    const int co = e / 10, g = e - co * 10;
    uint4 w = make_uint4(0, 0, 0, 0);
    if (j0 + co < p.N) w = *(const uint4*)(p.w + (int64_t)(j0 + co) * p.kf + g * 8);
    *(uint4*)&wl[co * WPITCH + g * 16] = w;
  }
  if (threadIdx.x < 64) bl[threadIdx.x] = j0 + (int)threadIdx.x < p.N ? p.bias[j0 + threadIdx.x] : 0.f;
  f32x16 acc[2][2];                                        // [32 pixels][32 channels]
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[a][b][e] = 0.f;
  __syncthreads();                                         // (the weights)
#pragma unroll
  for (int kk = 0; kk < 5; ++kk) {
    bf16x8 fa[2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int c = 0; c < 8; ++c) fa[a][c] = c < CIN ? (bf16)v[a][kk][c < CIN ? c : 0] : (bf16)0.f;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      if (b == 1 && !upper) continue;
      const bf16x8 fb = *(const bf16x8*)&wl[(b * 32 + l31) * WPITCH + (2 * kk + h) * 16];
#pragma unroll
      for (int a = 0; a < 2; ++a) acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb, fa[a], acc[a][b], 0, 0, 0);
    }
  }
  // accumulator element 4q + e of a lane: channel 8q + 4h + e, pixel l31
  char* const mine = area[wave];
  const uint4 keep = keep8(p.N - j0 - (lane & 7) * 8);
#pragma unroll
  for (int a = 0; a < 2; ++a) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      if (b == 1 && !upper) continue;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 bv = *(const f32x4*)&bl[b * 32 + 8 * q + 4 * h];
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float t = acc[a][b][4 * q + e] + bv[e];
          if (p.relu) t = fmaxf(t, 0.f);
          o[e] = (bf16)t;
        }
        *(bf16x4*)(mine + l31 * OPITCH + (b * 32 + 8 * q + 4 * h) * 2) = o;
      }
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int t = 0; t < 4; ++t) {                          // (channels past N, which nothing has written here: zeros)
      const int r = 8 * t + (lane >> 3);
      const int64_t pix = pix0 + a * 32 + r;
      const uint4 o = *(const uint4*)(mine + r * OPITCH + (lane & 7) * 16);
      if (pix < p.pixels && j0 + (lane & 7) * 8 < p.ldo) *(uint4*)(p.out + pix * p.ldo + j0 + (lane & 7) * 8) = o & keep;
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// Weight gradient.  A workgroup takes one chunk of a worker's pixels and 64 output channels.  A stage
// is 64 pixels: the dy rows (8 KB, global -> LDS, two stages ahead) and the transposed patches
// [tap * CIN + ci][pixel], built from values fetched a stage ahead; row 9 CIN holds ones, so that its
// result is the bias gradient.  Wave (wco, ks): 32 output channels, every other 16-pixel step; the two
// waves of a channel half add their results at the end.
constexpr int ROWS_P = 144;                // bytes per patch row
constexpr int DY_STAGE = 64 * 128;
constexpr int PART = 2 * 16 * 64;          // floats of a chunk result: [channel half][4 quads][lane] x 4

template <int CIN>
__global__ __launch_bounds__(256) void stem_wgrad_kernel(StemArgs p, Segs segs, RowChunks ch) {
  __shared__ __align__(16) uint4 dyring[3 * DY_STAGE / 16];
  __shared__ __align__(16) char patch[2][32 * ROWS_P];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int chunk = blockIdx.x, cob = blockIdx.y;
  int k = 0;
  while (k + 1 < segs.K && chunk >= ch.first[k + 1]) ++k;
  const int r0 = segs.off[k] + (chunk - ch.first[k]) * ch.rows;
  const int n = min(ch.rows, segs.off[k + 1] - r0);
  const int T = (n + 63) / 64;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)&dyring[0];

  // rows of the patches that no tap fills: ones, then zeros
  for (int e = tid; e < 2 * (32 - 9 * CIN) * 64; e += 256) {
    const int b = e / ((32 - 9 * CIN) * 64), in = e - b * (32 - 9 * CIN) * 64, row = 9 * CIN + (in >> 6);
    *(bf16*)&patch[b][row * ROWS_P + (in & 63) * 2] = (bf16)(row == 9 * CIN ? 1.f : 0.f);
  }
  // dy: copy c = wave + 4u moves pixels 8c .. 8c+7; the 64-byte halves of pixels 2, 3, 6, 7, ... swapped
  const int dslot = 8 * wave + (lane >> 3);
  const int dg = (lane & 7) ^ (((dslot >> 1) & 1) << 2);
  const char* dsrc = (const char*)(p.dy + (int64_t)(r0 + dslot) * p.ldd + cob * 64 + dg * 8);
  const int64_t dpix = p.ldd * 2;
  int dleft = cob * 64 + dg * 8 < p.ldd ? n - dslot : 0;   // (a narrow row has no upper half: zeros)
  auto issue = [&](uint32_t base) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
      async_copy_1k(dleft > 32 * u ? (const void*)(dsrc + u * 32 * dpix) : p.zeros,
                    base + (uint32_t)((wave + 4 * u) * 1024));
    dsrc += 64 * dpix;
    dleft -= 64;
  };
  // patches: this thread gathers pixel tid % 64 under the taps part, part + 4, part + 8
  const int part = tid >> 6;
  int at = lane, row = (r0 + lane) / p.Wo, ox = (r0 + lane) - row * p.Wo, img = row / p.Ho, oy = row - img * p.Ho;
  float v[3][CIN];
  auto gather = [&]() {                    // the next stage's pixel
#pragma unroll
    for (int i = 0; i < 3; ++i) fetch_tap<CIN>(p, img, oy, ox, part + 4 * i, at < n && part + 4 * i < 9, v[i]);
    at += 64;
    ox += 64;
    while (ox >= p.Wo) { ox -= p.Wo; ++oy; }
    while (oy >= p.Ho) { oy -= p.Ho; ++img; }
  };
  auto put = [&](int b) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const int tap = part + 4 * i;
      if (tap >= 9) continue;
#pragma unroll
      for (int c = 0; c < CIN; ++c) *(bf16*)&patch[b][(tap * CIN + c) * ROWS_P + lane * 2] = (bf16)v[i][c];
    }
  };

  const int wco = wave & 1, ks = wave >> 1, l31 = lane & 31, h = lane >> 5;
  const int g = lane >> 4, r = lane & 15;
  const uint32_t foff = (uint32_t)((8 * (g >> 1) + (r >> 2)) * 128 + ((wco ^ ((r >> 3) & 1)) * 64) +
                                   (16 * (g & 1) + 4 * (r & 3)) * 2);
  f32x16 acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
  gather();
#pragma unroll 1
  for (int t = 0; t < 2 && t < T; ++t) issue(lds0 + (uint32_t)(t * DY_STAGE));
  uint32_t buf = lds0, nbuf = lds0 + 2 * DY_STAGE;
  for (int t = 0; t < T; ++t) {
    put(t & 1);                            // (its values were asked for before the copies still pending)
    if (t + 1 < T) asm volatile("s_waitcnt vmcnt(2)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();                       // stage t visible; stage t-1 no longer read
    if (t + 1 < T) gather();
    if (t + 2 < T) issue(nbuf);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int step = 2 * s + ks;
      const uint32_t a = buf + foff + (uint32_t)(step * 16 * 128);
      const s16x4 lo = lds_read_tr(a), hi = lds_read_tr(a + 4 * 128);
      const s16x8 d = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      const bf16x8 x8 = *(const bf16x8*)&patch[t & 1][l31 * ROWS_P + (step * 16 + 8 * h) * 2];
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, d), x8, acc, 0, 0, 0);
    }
    buf = buf == lds0 + 2 * DY_STAGE ? lds0 : buf + DY_STAGE;
    nbuf = nbuf == lds0 + 2 * DY_STAGE ? lds0 : nbuf + DY_STAGE;
  }
  // the two waves of a channel half: ks = 0 plus ks = 1
  __syncthreads();
  f32x4* const area = (f32x4*)&dyring[0];
  if (ks == 1) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      area[(wco * 4 + q) * 64 + lane] = f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
  }
  __syncthreads();
  if (ks == 0) {
    f32x4* const out = (f32x4*)(p.partial + ((int64_t)chunk * gridDim.y + cob) * PART);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      out[(wco * 4 + q) * 64 + lane] =
          f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]} + area[(wco * 4 + q) * 64 + lane];
  }
}

// Worker k's chunk results added in a fixed order.  256 threads = 32 quads x 8 chunk-lanes.  Quad
// (channel half, q, lane) of a chunk: patch row lane % 32, channels 8q + 4 (lane / 32) .. of the half.
__global__ __launch_bounds__(256) void stem_reduce_kernel(const float* __restrict__ partial, int rows, int Cout,
                                                          float* __restrict__ dW, float* __restrict__ db,
                                                          int64_t group_stride, RowChunks ch) {
  __shared__ f32x4 red[8][32];
  const int il = threadIdx.x & 31, q8 = threadIdx.x >> 5, k = blockIdx.y;
  const int cobs = (Cout + 63) / 64, cob = blockIdx.x / (PART / 128), idx = (blockIdx.x % (PART / 128)) * 32 + il;
  const f32x4* src = (const f32x4*)partial + (int64_t)cob * (PART / 4) + idx;
  const int64_t stride = (int64_t)cobs * (PART / 4);
  // (four independent partial sums, so that the loads overlap)
  const int last = ch.first[k + 1];
  f32x4 a0 = {0.f, 0.f, 0.f, 0.f}, a1 = a0, a2 = a0, a3 = a0;
  int c = ch.first[k] + q8;
  for (; c + 24 < last; c += 32) {
    a0 += src[c * stride];
    a1 += src[(c + 8) * stride];
    a2 += src[(c + 16) * stride];
    a3 += src[(c + 24) * stride];
  }
  for (; c < last; c += 8) a0 += src[c * stride];
  f32x4 sum = (a0 + a1) + (a2 + a3);
  red[q8][il] = sum;
  __syncthreads();
  if (q8 != 0) return;
#pragma unroll
  for (int i = 1; i < 8; ++i) sum += red[i][il];
  const int lane = idx & 63, m = lane & 31, co = cob * 64 + (idx >> 8) * 32 + 8 * ((idx >> 6) & 3) + 4 * (lane >> 5);
  if (m > rows) return;
  float* dst = m == rows ? db + (int64_t)k * group_stride + co : dW + (int64_t)k * group_stride + (int64_t)m * Cout + co;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (co + e < Cout) dst[e] = sum[e];
}

}  // namespace

bool conv_stem_applies(int Cin) { return Cin <= 3; }

int launch_stem_forward(const float* x, int Cin, int H, int W, int Ho, int Wo, int stride, int64_t pixels,
                        const void* w, int kf, const float* bias, int N, int relu, void* out,
                        int64_t ldo, double flops, double bytes, void* stream) {
  if (Cin < 1 || Cin > 3 || kf < 80 || kf % 8 || ldo % 32 || ldo < N || pixels >= (int64_t)1 << 31 ||
      (((uintptr_t)w | (uintptr_t)out) & 15))
    return fail(DYNB_ERR_BADARG, "stem: one to three channels, whole 32-channel blocks");
  if (pixels == 0) return DYNB_OK;
  StemArgs p = {};
  p.x = x; p.H = H; p.W = W; p.Ho = Ho; p.Wo = Wo; p.stride = stride; p.pixels = pixels;
  p.w = (const bf16*)w; p.kf = kf; p.bias = bias; p.N = N; p.relu = relu;
  p.out = (bf16*)out; p.ldo = ldo;
  Timed t(KC_GEMM_FWD, stream, flops, bytes);
  const dim3 grid((unsigned)((pixels + 255) / 256), (unsigned)((ldo + 63) / 64));
  const hipStream_t st = (hipStream_t)stream;
  if (Cin == 1) hipLaunchKernelGGL(stem_forward_kernel<1>, grid, dim3(256), 0, st, p);
  else if (Cin == 2) hipLaunchKernelGGL(stem_forward_kernel<2>, grid, dim3(256), 0, st, p);
  else hipLaunchKernelGGL(stem_forward_kernel<3>, grid, dim3(256), 0, st, p);
  return hipGetLastError() == hipSuccess ? DYNB_OK : fail(DYNB_ERR_HIP, "stem: launch failed");
}

int launch_stem_wgrad(const float* x, int Cin, int H, int W, int Ho, int Wo, int stride, const void* dy,
                      int64_t ldd, int Cout, int chunk_rows, float* scratch, int64_t scratch_floats, float* dW,
                      float* db, int64_t group_stride, const Segs& s, double flops, double bytes, void* stream) {
  const int cobs = (Cout + 63) / 64;
  if (Cin < 1 || Cin > 3 || ldd % 32 || ldd < Cout || chunk_rows < 64 ||
      (((uintptr_t)dy | (uintptr_t)scratch) & 15))
    return fail(DYNB_ERR_BADARG, "stem: one to three channels, whole 32-channel blocks, 16-byte aligned");
  const RowChunks ch = make_row_chunks(s, chunk_rows);
  const int nch = ch.first[s.K];
  if ((int64_t)nch * cobs * PART > scratch_floats) return fail(DYNB_ERR_BADARG, "stem: scratch area too small");
  StemArgs p = {};
  p.x = x; p.H = H; p.W = W; p.Ho = Ho; p.Wo = Wo; p.stride = stride; p.pixels = s.off[s.K];
  p.dy = (const bf16*)dy; p.ldd = ldd; p.partial = scratch;
  p.zeros = device_zero_granule();
  if (!p.zeros) return fail(DYNB_ERR_HIP, "stem: no address for the zero granule");
  Timed t(KC_GEMM_WGRAD, stream, flops, bytes);
  const dim3 grid(nch, cobs);
  const hipStream_t st = (hipStream_t)stream;
  if (nch > 0) {
    if (Cin == 1) hipLaunchKernelGGL(stem_wgrad_kernel<1>, grid, dim3(256), 0, st, p, s, ch);
    else if (Cin == 2) hipLaunchKernelGGL(stem_wgrad_kernel<2>, grid, dim3(256), 0, st, p, s, ch);
    else hipLaunchKernelGGL(stem_wgrad_kernel<3>, grid, dim3(256), 0, st, p, s, ch);
  }
  hipLaunchKernelGGL(stem_reduce_kernel, dim3((unsigned)(cobs * (PART / 128)), s.K), dim3(256), 0, st, scratch,
                     9 * Cin, Cout, dW, db, group_stride, ch);
  return hipGetLastError() == hipSuccess ? DYNB_OK : fail(DYNB_ERR_HIP, "stem: launch failed");
}

}  // namespace dynb
