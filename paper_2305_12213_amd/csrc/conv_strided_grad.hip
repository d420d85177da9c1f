// Input gradient of a 3x3 convolution with stride 2 and zero padding 1 (bf16 NHWC), up to 128 channels on the
// side of dy, dy images up to 64 pixels wide.
//
// dy pixel (a, b) and its neighbours to the right and below determine the four input pixels (2a, 2b) ..
// (2a + 1, 2b + 1): an input pixel of even row and column is reached by one tap, of odd row or column by two,
// of both by four -- nine products for four pixels.  The dy pixels of all images are one flat run; a
// workgroup takes 256 of them and 32 input channels, copies the run that they and their neighbours span (256 +
// width + 1 pixels) and the nine taps' weights into LDS once, and reads all operands from there; neighbours
// outside the image are read from a pixel of zeros.  A step of 16 channels is 18 matrix instructions of a
// wave on 17 operands.
// The gathered-operand product, one launch part per parity class, fetches dy 2.25 times, fills half of its 64
// columns where there are 32 channels, and starts and ends a pipeline for every 64 to 512 reduction indices:
// 512 x 16 x 16, 64 -> 32 channels of 32 x 32: 49 -> 25 us (84 MB: 3.4 TB/s); 512 x 8 x 8, 128 -> 64: 22 -> 20, one workgroup's
// way in and out on every compute unit.
#include <hip/hip_runtime.h>

#include "device_rows.h"
#include "dynb_internal.h"
#include "lds_async.h"

namespace dynb {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int MAX_W = 64;
constexpr int CELLS = 256;                             // dy pixels per workgroup, 64 per wave

struct StridedGradArgs {
  const bf16* dy; int64_t ldd;       // [images * Ho * Wo][ldd]
  const bf16* w; int64_t ldw;        // [N][ldw]: w[j][tap * cp + c]
  int Ho, Wo, H, W, total;           // total: dy pixels
  int cp, N;                         // channels per tap (a multiple of 8), input channels
  bf16* out; int64_t ldo;            // [images * H * W][ldo]
  const bf16* mask; int64_t ldmask;  // zero where mask <= 0 (optional)
  const bf16* addend; int64_t ldadd; // added after rounding (optional)
  const void* zeros;
};

// RB: bytes of LDS per pixel and per weight row: 64, 128 or 256 for up to 32, 64 or 128 channels
template <int RB>
struct StridedGrad {
  static constexpr int G = RB / 16;                    // granules
  static constexpr int HALO = (CELLS + MAX_W + 1) * RB;
  static constexpr int HALO_AREA = (HALO + 1023) / 1024 * 1024;
  static constexpr int WEIGHTS = 9 * 32 * RB;          // [tap][input channel]
  static constexpr int ZEROS = HALO_AREA + WEIGHTS;
  static constexpr int OPITCH = 144;                   // bytes per cell of the result patch: two pixels x 32 channels
  static constexpr int AREA = ZEROS + RB > 4 * 64 * OPITCH ? ZEROS + RB : 4 * 64 * OPITCH;
  static_assert(AREA <= 160 * 1024 && WEIGHTS % 1024 == 0, "LDS");
};

// Granule g of row r sits at slot g ^ swz(r): 16 neighbouring rows at one granule take all 64 banks.
template <int RB>
__device__ inline int swz(int r) {
  return RB == 256 ? r & 15 : RB == 128 ? swizzle128(r) : (((r >> 2) & 1) << 1) | ((r >> 3) & 1);
}

template <int RB>
__global__ __launch_bounds__(256, RB == 256 ? 1 : 2) void conv_strided_grad_kernel(StridedGradArgs p) {
  using F = StridedGrad<RB>;
  __shared__ __align__(256) char area[F::AREA];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l31 = lane & 31, h = lane >> 5;
  const int p0 = blockIdx.x * CELLS, j0 = blockIdx.y * 32;
  const uint32_t lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)&area[0];
  if (threadIdx.x < F::G) *(uint4*)&area[F::ZEROS + threadIdx.x * 16] = make_uint4(0, 0, 0, 0);

  // ---- copies: 1 KB = 64 / G rows; pixels past the batch and channels past cp are zeros
  constexpr int RPC = 64 / F::G;
  const int cg = p.cp / 8, halo = CELLS + p.Wo + 1;
#pragma unroll 1
  for (int c = wave; c * RPC < halo; c += 4) {
    const int r = c * RPC + lane / F::G, g = (lane % F::G) ^ swz<RB>(r);
    const bool ok = p0 + r < p.total && g < cg;
    async_copy_1k(ok ? (const void*)(p.dy + (int64_t)(p0 + r) * p.ldd + g * 8) : p.zeros, lds + (uint32_t)(c * 1024));
  }
#pragma unroll 1
  for (int c = wave; c * RPC < 9 * 32; c += 4) {
    const int r = c * RPC + lane / F::G, tap = r >> 5, j = j0 + (r & 31), g = (lane % F::G) ^ swz<RB>(r & 31);
    const bool ok = j < p.N && g < cg;
    async_copy_1k(ok ? (const void*)(p.w + (int64_t)j * p.ldw + tap * p.cp + g * 8) : p.zeros,
                  lds + (uint32_t)(F::HALO_AREA + c * 1024));
  }

  // ---- where this lane's two cells and their neighbours lie: [cell][right + 2 below], granule h
  uint32_t at[2][4];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int r = wave * 64 + s * 32 + l31, i = p0 + r < p.total ? p0 + r : 0;
    const int yy = i / p.Wo, x = i - yy * p.Wo, y = yy % p.Ho;
    const bool right = x + 1 < p.Wo, below = y + 1 < p.Ho;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int n = r + (q & 1) + (q >> 1) * p.Wo;
      const bool ok = (!(q & 1) || right) && (!(q >> 1) || below);
      at[s][q] = ok ? (uint32_t)(n * RB + ((h ^ swz<RB>(n)) * 16)) : (uint32_t)F::ZEROS;
    }
  }
  const uint32_t wat = (uint32_t)(F::HALO_AREA + l31 * RB + ((h ^ swz<RB>(l31)) * 16));

  f32x16 acc[4][2];                                    // [class: odd column + 2 odd row][cell]
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[c][s][v] = 0.f;

  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  const int steps = (p.cp + 15) / 16;
#pragma unroll 1
  for (int k = 0; k < steps; ++k) {
    const uint32_t x = (uint32_t)(k * 32);             // (granule 2k + h: the slots are xors)
    bf16x8 fa[2][4];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q) fa[s][q] = *(const bf16x8*)(area + (at[s][q] ^ x));
    // tap (kh, kw) leads from neighbour (kh == 0 below, kw == 0 right) to the class (kh != 1, kw != 1)
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      const int kh = tap / 3, kw = tap % 3, c = (kw != 1 ? 1 : 0) + (kh != 1 ? 2 : 0), q = (kw == 0 ? 1 : 0) + (kh == 0 ? 2 : 0);
      const bf16x8 fb = *(const bf16x8*)(area + ((wat + (uint32_t)(tap * 32 * RB)) ^ x));
#pragma unroll
      for (int s = 0; s < 2; ++s) acc[c][s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb, fa[s][q], acc[c][s], 0, 0, 0);
    }
  }
  __syncthreads();                                     // (the patches overwrite what was read)

  // ---- results, one row of input pixels at a time: through the wave's patch, so that a lane stores 16 bytes of
  // a pixel and eight lanes the two neighbouring pixels of a cell.  Accumulator element 4t + e: channel 8t +
  // 4h + e, cell l31.
  char* const patch = area + wave * 64 * F::OPITCH;
  const int part = lane & 7, px = part >> 2, ch = (part & 3) * 8;
  const uint4 keep = keep8(p.N - j0 - ch);
  int pixel[8];                                        // of row 0 of cell 8t + lane / 8, -1: none
  uint32_t odd_row = 0;                                // bit t: its row 1 exists
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    const int i = p0 + wave * 64 + 8 * t + (lane >> 3), ic = i < p.total ? i : 0;
    const int yy = ic / p.Wo, b = ic - yy * p.Wo, n = yy / p.Ho, a = yy - n * p.Ho;
    const bool ok = i < p.total && 2 * b + px < p.W;
    pixel[t] = ok ? (n * p.H + 2 * a) * p.W + 2 * b + px : -1;
    if (ok && 2 * a + 1 < p.H) odd_row |= 1u << t;
  }
#pragma unroll
  for (int py = 0; py < 2; ++py) {
    uint4 mk[8], ad[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const bool ok = py == 0 ? pixel[t] >= 0 : (odd_row >> t) & 1u;
      const int64_t i = ok ? pixel[t] + py * p.W : 0;  // (pixel 0 where there is none)
      if (p.mask) mk[t] = load8(p.mask + i * p.ldmask + j0 + ch);
      if (p.addend) ad[t] = load8(p.addend + i * p.ldadd + j0 + ch);
    }
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          bf16x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = (bf16)acc[2 * py + c][s][4 * t + e];
          *(bf16x4*)(patch + (s * 32 + l31) * F::OPITCH + c * 64 + (8 * t + 4 * h) * 2) = o;
        }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      uint4 v = *(const uint4*)(patch + (8 * t + (lane >> 3)) * F::OPITCH + part * 16);
      if (p.addend) {
        float f[8], d[8];
        unpack8(v, f);
        unpack8(ad[t], d);
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] += d[e];
        v = pack8(f);
      }
      if (p.mask) {
        v = v & positive8(mk[t]);
      }
      if (py == 0 ? pixel[t] >= 0 : (odd_row >> t) & 1u)
        store8(p.out + (int64_t)(pixel[t] + py * p.W) * p.ldo + j0 + ch, v & keep);
    }
    __builtin_amdgcn_wave_barrier();
  }
}

}  // namespace

// Where it is faster than the gathered-operand product: 11030 calls of 1 to 700 images of 4 x 4 to 64 x 64 pixels,
// 4 to 512 input channels, 8 to 128 on the side of dy, timed on both (launch and its events, us; the product's
// time first).  A launch runs in rounds of 512 workgroups (256 with more than 64 channels on the side of dy), and every
// further 32 input channels copy the same run again; the product's tiles are 64 columns wide, 128 for more than 64.
//   up to 64 input channels: everywhere (32 x 32 pixels, 512 images, 32 -> 24 channels 47, 24; 64 images, 64 -> 64 16.0,
//     15.0) but for the smallest launches of few channels (4 x 4, 64 images, 64 -> 8: 11.6, 12.2);
//   more: where the product's last tile of columns is at most three quarters full (28 x 28, 96 images, 96 -> 40:
//     22, 17), unless a second round is just begun (16 x 16, 700 images, 72 -> 40, 525 workgroups: 33, 38); otherwise
//     in one round or in whole ones (9 x 64, 160 images, 128 -> 8, 400 workgroups: 20.0, 19.3; 16 x 16, 256 images,
//     512 -> 24, 1024: 47, 34; but 700 images, 128 -> 8, 700: 30, 37);
//   more than 64 channels of dy: up to 32 input channels, above the smallest launches (64 x 64, 64 images, 32 -> 128: 37,
//     21); more, only in one nearly full round (16 x 16, 512 images, 64 -> 128: 23.0, 22.4; 700 images 33, 37; 13 x 21,
//     160 images, 256 -> 96: 28, 35).
static bool faster_than_gathered(int cp, int N, int64_t blocks) {
  const bool loose = N % 128 >= 1 && N % 128 <= 96;    // (columns of the product's last tile)
  if (cp > 64) return N <= 32 ? N <= 16 || blocks >= 96 : loose && blocks > 192 && blocks <= 256;
  if (N <= 64) return N <= 16 || cp >= 48 || blocks >= 96;
  if (loose) return blocks > 192 && (blocks <= 512 || blocks >= 560);
  return blocks > 256 && (blocks <= 512 || blocks % 512 == 0 || blocks % 512 >= 496);
}

bool conv_strided_grad_applies(int dtype, const GemmArgs& a) {
  if (dtype != DYNB_BF16 || a.conv != 2 || a.mode != MODE_DGRAD || a.stride != 2 || a.Cf || !a.C) return false;
  if (a.cp > 128 || a.src_w > MAX_W || a.src_h != (a.row_h + 1) / 2 || a.src_w != (a.row_w + 1) / 2) return false;
  const int64_t block = round_up(a.N, 32);             // the channels that whole blocks cover
  if (a.M % (a.row_h * a.row_w) || a.lda < a.cp || a.lda % 8 || a.ldb < 9 * a.cp || a.ldb % 8) return false;
  if (a.ldc < block || a.ldc % 8 || (a.mask && (a.ldmask < block || a.ldmask % 8))) return false;
  if (a.addend && (a.ldadd < block || a.ldadd % 8)) return false;
  const int64_t cells = (int64_t)(a.M / (a.row_h * a.row_w)) * a.src_h * a.src_w;
  return faster_than_gathered(a.cp, a.N, (cells + CELLS - 1) / CELLS * (block / 32));
}

int launch_conv_strided_grad(const GemmArgs& a, void* stream) {
  StridedGradArgs p = {};
  p.zeros = device_zero_granule();
  if (!p.zeros) return fail(DYNB_ERR_HIP, "conv_strided_grad: no address for the zero granule");
  p.dy = (const bf16*)a.A; p.ldd = a.lda;
  p.w = (const bf16*)a.B; p.ldw = a.ldb;
  p.Ho = a.src_h; p.Wo = a.src_w; p.H = a.row_h; p.W = a.row_w;
  p.total = a.M / (a.row_h * a.row_w) * a.src_h * a.src_w;
  p.cp = a.cp; p.N = a.N;
  p.out = (bf16*)a.C; p.ldo = a.ldc;
  p.mask = (const bf16*)a.mask; p.ldmask = a.ldmask;
  p.addend = (const bf16*)a.addend; p.ldadd = a.ldadd;
  const auto kernel = a.cp <= 32 ? conv_strided_grad_kernel<64> : a.cp <= 64 ? conv_strided_grad_kernel<128>
                                                                             : conv_strided_grad_kernel<256>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)((p.total + CELLS - 1) / CELLS), (unsigned)((a.N + 31) / 32)), dim3(256), 0,
                     (hipStream_t)stream, p);
  return hipGetLastError() == hipSuccess ? DYNB_OK : fail(DYNB_ERR_HIP, "conv_strided_grad: launch failed");
}

}  // namespace dynb
