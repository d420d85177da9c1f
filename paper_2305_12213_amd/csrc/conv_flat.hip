// 3x3 convolution, stride 1, zero padding 1, on images up to 64 pixels wide, for up to 64 reduction
// channels (bf16 NHWC): forward and input gradient from one halo run in LDS.
//
// The pixels of all images are one flat run.  A workgroup takes 64 consecutive output pixels per wave,
// copies the run that they and their neighbours one image row up and down span (64 waves + 2 W + 2
// pixels) and the weights of its output channels into LDS, once, and reads every tap's operand from
// there at a pixel offset; a tap that falls outside the image reads a pixel of zeros instead.  The
// gathered-operand GEMM, which serves the shapes that this kernel does not take, copies a shifted tile
// of its own for each tap, with an address per copy and lane, and pads narrow outputs to 64 channels.
// The reduction runs through (tap, channel) as the weights lie in memory, 16 at a time -- a step may
// span two taps, the two lane halves then work on different ones -- so sums keep the GEMM's order.
// Launches are a few microseconds long: loops are rolled, as code is fetched at about 2 KB/us.
// 167 x 28 x 28 pixels, 24 -> 24 channels: forward 18 -> 11 us, input gradient 24 -> 13;
// 367 x 28 x 28, 24 -> 64 and 64 -> 24: 41 and 52 -> 32 and 39.  Bias, mask and addend asked for along with the copies
// instead of value by value at the end: 24 -> 24 forward 10.5 -> 9.5, input gradient with a mask 12.2 -> 11.  (Operands of
// the next step fetched ahead, two register sets: slower, models of up to 32 channels 3 % on average.)
#include <hip/hip_runtime.h>

#include "device_rows.h"
#include "dynb_internal.h"
#include "lds_async.h"

namespace dynb {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int MAX_W = 64;

struct ConvFlatArgs {
  const bf16* src; int64_t lds;      // [total][lds]
  const bf16* w; int64_t ldw;        // [N][ldw]: w[j][tap * cp + c], ldw a multiple of 64
  int W, H, total;                   // image sides, pixels of the batch
  int cp, N;                         // channels per tap (a multiple of 8), output channels
  int flip;                          // 0: tap (kh, kw) reads pixel (y + kh - 1, x + kw - 1); 1: (y + 1 - kh, ...)
  const float* bias; int relu;       // forward
  bf16* out; int64_t ldo;
  const bf16* mask; int64_t ldmask;  // input gradient: zero where mask <= 0 (optional)
  const bf16* addend; int64_t ldadd; // input gradient: added after rounding (optional)
  const void* zeros;
};

// CI / CO: 32-channel blocks of the reduction and the output side; NW waves.
template <int CI, int CO, int NW>
struct FlatConv {
  static constexpr int RB = 64 * CI;                          // bytes per halo pixel
  static constexpr int PIX = 64 * NW + 2 * MAX_W + 2;
  static constexpr int HALO = (PIX * RB + 1023) / 1024 * 1024;
  static constexpr int MAX_KF = CI == 1 ? 320 : 576;          // reduction length, padded to 64
  static constexpr int WEIGHTS = 32 * CO * MAX_KF * 2;
  static constexpr int OPITCH = 64 * CO + 16;                 // bytes per pixel of the result patch
  static constexpr int AREA = HALO + WEIGHTS + RB;            // ... and a pixel of zeros
  static_assert(NW * 64 * OPITCH <= AREA && AREA <= 160 * 1024, "LDS");
};

// Granule g of halo row r sits at slot g ^ swz(r): 16 neighbouring rows at one granule take all 64 banks.
template <int CI>
__device__ inline int swz(int r) {
  return CI == 2 ? swizzle128(r) : (((r >> 2) & 1) << 1) | ((r >> 3) & 1);
}

template <int CI, int CO, int NW>
__global__ __launch_bounds__(NW * 64) void conv_flat_kernel(ConvFlatArgs p) {
  using F = FlatConv<CI, CO, NW>;
  __shared__ __align__(16) char area[F::AREA];
  __shared__ __align__(16) float bias[32 * CO];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l31 = lane & 31, h = lane >> 5;
  const int p0 = blockIdx.x * (64 * NW), j0 = blockIdx.y * (32 * CO);
  const uint32_t lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)&area[0];
  const uint32_t lds_w = lds + F::HALO;
  if (threadIdx.x < F::RB / 16) *(uint4*)&area[F::HALO + F::WEIGHTS + threadIdx.x * 16] = make_uint4(0, 0, 0, 0);

  // ---- copies: halo pixel r is pixel p0 - W - 1 + r of the batch (zeros outside it)
  constexpr int GP = 4 * CI;                           // granules per pixel
  const int halo = 64 * NW + 2 * p.W + 2;
  for (int c = wave; c * (64 / GP) < halo; c += NW) {
    const int r = c * (64 / GP) + lane / GP, s = p0 - p.W - 1 + r, g = (lane % GP) ^ swz<CI>(r);
    const bool ok = s >= 0 && s < p.total;
    async_copy_1k(ok ? (const void*)(p.src + (int64_t)s * p.lds + g * 8) : p.zeros, lds + (uint32_t)(c * 1024));
  }
  // weights: rows of kf / 8 granules, granule g of row r at slot g ^ (r % 8); channels past the last
  // are zeros
  const int gw = (int)(p.ldw / 8);
  for (int c = wave; c * 64 < 32 * CO * gw; c += NW) {
    const int s = c * 64 + lane, r = s / gw, g = (s - r * gw) ^ (r & 7);
    const bool ok = r < 32 * CO && j0 + r < p.N;
    async_copy_1k(ok ? (const void*)(p.w + (int64_t)(j0 + r) * p.ldw + g * 8) : p.zeros, lds_w + (uint32_t)(c * 1024));
  }

  // ---- what the end needs, asked for now: the bias, and the mask and addend rows of this lane's results (rows past
  // the last repeat it)
  constexpr int LPR = 4 * CO, RPI = 64 / LPR;          // lanes per row of a wave's results, rows per instruction
  const int ch = (lane % LPR) * 8;
  float mine = 0.f;
  if (threadIdx.x < 32 * CO && p.bias && j0 + (int)threadIdx.x < p.N) mine = p.bias[j0 + threadIdx.x];
  bf16x8 addend[LPR], mask[LPR];
#pragma unroll
  for (int t = 0; t < LPR; ++t) {
    const int64_t i = min(p0 + wave * 64 + t * RPI + lane / LPR, p.total - 1);
    if (p.addend) addend[t] = *(const bf16x8*)(p.addend + i * p.ldadd + j0 + ch);
    if (p.mask) mask[t] = *(const bf16x8*)(p.mask + i * p.ldmask + j0 + ch);
  }

  // ---- this lane's two pixels: which of the nine neighbours lie inside the image
  int row[2];
  uint32_t in[2];
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    row[a] = wave * 64 + a * 32 + l31;
    const int q = p0 + row[a] < p.total ? p0 + row[a] : 0, yy = q / p.W, x = q - yy * p.W, y = yy % p.H;
    uint32_t m = 0x1ff;
    if (y == 0) m &= ~0x007u;
    if (y == p.H - 1) m &= ~0x1c0u;
    if (x == 0) m &= ~0x049u;
    if (x == p.W - 1) m &= ~0x124u;
    in[a] = m;
  }
  f32x16 acc[2][CO];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < CO; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

  if (threadIdx.x < 32 * CO) bias[threadIdx.x] = mine;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  const int ng = p.cp / 8, steps = (9 * ng + 1) / 2;
  int tap = h / ng, q = h - tap * ng;                  // this lane half's granule 2 s + h: tap, granule in it
  const char* const wbase = area + F::HALO + l31 * (gw * 16);
#pragma unroll 1
  for (int s = 0; s < steps; ++s) {
    const int e = p.flip ? 8 - tap : tap, kh = (e * 11) >> 5;         // (e / 3 for 0 <= e < 9)
    const int shift = kh * p.W + e - 3 * kh;
    bf16x8 fa[2], fb[CO];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const int r = row[a] + shift;
      const bool ok = tap < 9 && ((in[a] >> (e & 31)) & 1u);
      const int at = ok ? r * F::RB + ((q ^ swz<CI>(r)) * 16) : F::HALO + F::WEIGHTS;
      fa[a] = *(const bf16x8*)(area + at);
    }
#pragma unroll
    for (int b = 0; b < CO; ++b)
      fb[b] = *(const bf16x8*)(wbase + b * 32 * gw * 16 + (((2 * s + h) ^ (l31 & 7)) * 16));
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < CO; ++b)
        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[b], fa[a], acc[a][b], 0, 0, 0);
    q += 2;
    if (q >= ng) { q -= ng; ++tap; }
    if (q >= ng) { q -= ng; ++tap; }
  }
  __syncthreads();                                     // the halo and the weights are no longer read

  // ---- results through LDS: a wave's 64 pixels, then whole rows of 64 or 128 bytes.  Accumulator
  // element 4t + e of a lane: channel 8t + 4h + e, pixel l31.
  char* const patch = area + wave * 64 * F::OPITCH;
#pragma unroll
  for (int b = 0; b < CO; ++b)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const f32x4 bv = *(const f32x4*)&bias[b * 32 + 8 * t + 4 * h];
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float v = acc[a][b][4 * t + e] + bv[e];
          if (p.relu) v = fmaxf(v, 0.f);
          o[e] = (bf16)v;
        }
        *(bf16x4*)(patch + (a * 32 + l31) * F::OPITCH + (b * 32 + 8 * t + 4 * h) * 2) = o;
      }
    }
  __builtin_amdgcn_wave_barrier();
  const uint4 keep = keep8(p.N - j0 - ch);
#pragma unroll
  for (int t = 0; t < LPR; ++t) {
    const int r = t * RPI + lane / LPR;
    const int64_t i = p0 + wave * 64 + r;
    if (i >= p.total) continue;
    bf16x8 v = *(const bf16x8*)(patch + r * F::OPITCH + ch * 2);
    if (p.addend) {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = (bf16)((float)v[e] + (float)addend[t][e]);
    }
    if (p.mask) {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (!((float)mask[t][e] > 0.f)) v[e] = (bf16)0.f;
    }
    store8(p.out + i * p.ldo + j0 + ch, __builtin_bit_cast(uint4, v) & keep);
  }
}

template <int CI, int CO, int NW>
void launch_as(const ConvFlatArgs& p, hipStream_t st) {
  const dim3 grid((unsigned)((p.total + 64 * NW - 1) / (64 * NW)), (unsigned)((p.N + 32 * CO - 1) / (32 * CO)));
  hipLaunchKernelGGL((conv_flat_kernel<CI, CO, NW>), grid, dim3(NW * 64), 0, st, p);
}

}  // namespace

// (Asked after the kernels with resident weights, which take 64 to more than 32 channels up to 43 pixels wide, and with
// halo tiles: 32-pixel-wide images with whole 64-channel blocks, up to 32 outputs here.  Beyond 43 pixels 64 to more than
// 32 channels stay on the gathered-operand product: 64 is a power of two, for which its addressing is cheap, and
// fills its tile.  Other numbers of channels are faster here: 367 x 28 x 28 pixels, 48 -> 48 forward and input gradient 49 us
// each against 59 and 61, 56 -> 56 53 against 64 and 67.  Whole blocks of output channels are stored.)
bool conv_flat_applies(int dtype, const GemmArgs& a) {
  if (dtype != DYNB_BF16 || !a.conv || a.mode == MODE_WGRAD || a.stride != 1) return false;
  if (a.src_w > MAX_W || a.src_w != a.row_w || a.src_h != a.row_h || a.cp > 64 || (a.cp == 64 && a.N > 32)) return false;
  if (a.Cf || !a.C || a.M % (a.src_h * a.src_w) || a.lda % 32 || a.ldc % 32 || a.ldb % 64) return false;
  const int64_t block = a.N <= 32 ? 32 : round_up(a.N, 64);   // the output channels that whole blocks cover
  if (a.ldc < block || (a.mask && (a.ldmask % 32 || a.ldmask < block))) return false;
  if (a.addend && (a.ldadd % 32 || a.ldadd < block)) return false;
  return a.ldb <= (a.cp <= 32 ? 320 : 576) && a.ldb >= 9 * a.cp && a.lda >= (a.cp <= 32 ? 32 : 64);
}

int launch_conv_flat(const GemmArgs& a, void* stream) {
  ConvFlatArgs p = {};
  p.zeros = device_zero_granule();
  if (!p.zeros) return fail(DYNB_ERR_HIP, "conv_flat: no address for the zero granule");
  p.src = (const bf16*)a.A; p.lds = a.lda;
  p.w = (const bf16*)a.B; p.ldw = a.ldb;
  p.W = a.src_w; p.H = a.src_h; p.total = a.M;
  p.cp = a.cp; p.N = a.N;
  p.flip = a.conv == 2;
  p.bias = a.mode == MODE_FWD ? a.bias : nullptr;
  p.relu = a.mode == MODE_FWD ? a.relu : 0;
  p.out = (bf16*)a.C; p.ldo = a.ldc;
  p.mask = a.mode == MODE_DGRAD ? (const bf16*)a.mask : nullptr; p.ldmask = a.ldmask;
  p.addend = a.mode == MODE_DGRAD ? (const bf16*)a.addend : nullptr; p.ldadd = a.ldadd;
  const hipStream_t st = (hipStream_t)stream;
  // up to 32 channels on both sides three workgroups of four waves share a compute unit; 64-channel
  // weights leave room for one of eight
  if (a.cp <= 32 && a.N <= 32) launch_as<1, 1, 4>(p, st);
  else if (a.cp <= 32) launch_as<1, 2, 4>(p, st);
  else if (a.N <= 32) launch_as<2, 1, 8>(p, st);
  else launch_as<2, 2, 8>(p, st);
  return hipGetLastError() == hipSuccess ? DYNB_OK : fail(DYNB_ERR_HIP, "conv_flat: launch failed");
}

}  // namespace dynb
