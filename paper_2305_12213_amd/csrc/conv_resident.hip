// 3x3 convolution, stride 1, zero padding 1, 64 reduction channels, on images up to 43 pixels wide (bf16
// NHWC): forward and input gradient with the weights resident in LDS.
//
// A workgroup stays on its compute unit, keeps the 72 KB of weights of its 64 output channels in LDS and
// walks a run of tiles of 256 consecutive pixels (the pixels of all images are one flat run; a tap that
// falls outside the image reads a pixel of zeros).  Its eight waves are two groups of four, one wave of
// each on every SIMD, that take turns: while one group computes a tile -- nine taps read at pixel offsets
// from the halo run in LDS, no barrier in between -- the other writes its last tile out and fetches the
// halo of its next one.  The halo-tile kernel that streams the weights for every tile copies 116
// KB into LDS per tile instead of 41 and overlaps the phases of two workgroups only by chance.
// Sums run in the order of the other kernels: taps ascending, 16 channels at a time.
// 512 x 32 x 32 pixels, 64 -> 64 channels, as they run in a residual model: forward 41 us, input gradient with a mask
// 48 - 50, with mask and addend 61 - 63 (201 and 268 MB: 4.1 and 4.3 TB/s), 48 on average; the halo-tile kernel 58.
// Without the halo copies the forward takes as long, with a ninth of the matrix steps 31 us: a wave reads one operand
// from LDS per matrix instruction, 128 bytes per clock and compute unit, which is what the LDS delivers.
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
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int TILE = 256;                  // pixels
constexpr int HALO_COPIES = 43;            // 1 KB = 8 pixels each
constexpr int MAX_W = (HALO_COPIES * 8 - TILE - 2) / 2;
constexpr int HALO = HALO_COPIES * 1024;
constexpr int WEIGHTS = 9 * 64 * 128;      // [tap][output channel][64 channels]
constexpr int ZEROS = 2 * HALO + WEIGHTS;  // a pixel of zeros
constexpr int BIAS = ZEROS + 128;
constexpr int AREA = BIAS + 64 * 4;
constexpr int PER_WAVE = 11;               // halo copies of a wave, consecutive: the area under them is also the
constexpr int OPITCH = 144;                // wave's patch of results, 64 pixels of OPITCH bytes
static_assert(64 * OPITCH <= (HALO_COPIES - 3 * PER_WAVE) * 1024 && 4 * PER_WAVE >= HALO_COPIES, "patches");
static_assert(AREA <= 160 * 1024, "LDS");

struct ConvResidentArgs {
  const bf16* src; uint32_t pitch;   // [total], bytes per pixel
  uint32_t src_bytes, out_bytes;
  const bf16* w; uint32_t w_pitch;   // [N], bytes per output channel: tap * 128 + 2 channel
  int W, H, total, N;                // image sides, pixels of the batch, output channels
  int tiles;
  int flip;                          // 0: tap (kh, kw) reads pixel (y + kh - 1, x + kw - 1); 1: (y + 1 - kh, ...)
  const float* bias; int relu;       // forward
  bf16* out; uint32_t out_pitch;
  const bf16* mask; int64_t ldmask;  // input gradient: zero where mask <= 0 (optional)
  const bf16* addend; int64_t ldadd; // input gradient: added after rounding (optional)
};

template <bool MASK, bool ADD>
__global__ __launch_bounds__(512) void conv_resident_kernel(ConvResidentArgs p) {
  __shared__ __align__(128) char area[AREA];
  const int lane = threadIdx.x & 63, l31 = lane & 31, h = lane >> 5;
  const int wave8 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), group = wave8 >> 2, wave = wave8 & 3;
  const int j0 = blockIdx.y * 64;
  const uint32_t lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)&area[0];
  const int t0 = (int)((int64_t)p.tiles * blockIdx.x / gridDim.x);
  const int nt = (int)((int64_t)p.tiles * (blockIdx.x + 1) / gridDim.x) - t0;

  // ---- weights, a pixel of zeros, the bias (channels past the last are zeros)
  const i32x4 rsw = buffer_resource(p.w, (uint32_t)p.N * p.w_pitch);
#pragma unroll 1
  for (int c = wave8; c < 72; c += 8) {
    const int r = (c & 7) * 8 + (lane >> 3);
    async_copy_1k_buffer(rsw, (uint32_t)(j0 + r) * p.w_pitch + (uint32_t)((c >> 3) * 128 + ((lane & 7) ^ swizzle128(r)) * 16),
                         lds + 2 * HALO + (uint32_t)(c * 1024));
  }
  if (threadIdx.x < 8) *(uint4*)&area[ZEROS + threadIdx.x * 16] = make_uint4(0, 0, 0, 0);
  if (threadIdx.x < 64) {
    const int j = j0 + (int)threadIdx.x;
    *(float*)&area[BIAS + threadIdx.x * 4] = p.bias && j < p.N ? p.bias[j] : 0.f;
  }

  // ---- halo copies: pixel r of a tile's halo is pixel tile * 256 - W - 1 + r of the batch, zeros outside it
  // (the range check; a negative offset is a large one)
  const i32x4 rss = buffer_resource(p.src, p.src_bytes);
  const int copies = (TILE + 2 * p.W + 2 + 7) / 8;
  const int g_even = (lane & 7) ^ (((lane >> 4) & 3) << 1);    // granule for even copies, odd ones: its neighbour
  char* const halo = area + group * HALO;
  auto issue_halo = [&](int tile) {
    const uint32_t base = (uint32_t)(tile * TILE - p.W - 1 + (lane >> 3)) * p.pitch;
#pragma unroll 1
    for (int c = PER_WAVE * wave; c < PER_WAVE * (wave + 1) && c < copies; ++c)
      async_copy_1k_buffer(rss, base + (uint32_t)(8 * c) * p.pitch + (uint32_t)((g_even ^ (c & 1)) * 16),
                           lds + (uint32_t)(group * HALO + c * 1024));
  };

  // ---- a tile: this wave's 64 pixels x 64 channels
  f32x16 acc[2][2];
  uint4 mk[MASK ? 8 : 1], ad[ADD ? 8 : 1];
  uint32_t wat[4];                         // this lane's 16 bytes of weight row l31 in matrix step kk of a tap
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) wat[kk] = (uint32_t)(2 * HALO + l31 * 128 + (((2 * kk + h) ^ swizzle128(l31)) * 16));
  const int erow = lane >> 3, ecol = (lane & 7) * 8;       // results: this lane's row (of 8) and channels
  auto compute = [&](int tile) {
    const int p0 = tile * TILE + wave * 64;
    // (what the results will be combined with is on its way meanwhile)
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int i = p0 + 8 * t + erow;
      const int64_t ic = i < p.total ? i : p.total - 1;
      if constexpr (MASK) mk[t] = load8(p.mask + ic * p.ldmask + j0 + ecol);   // (rows are padded to 64 channels)
      if constexpr (ADD) ad[t] = load8(p.addend + ic * p.ldadd + j0 + ecol);
    }
    int row[2];
    uint32_t in[2];                        // which of the nine neighbours of this lane's pixels exist
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      row[a] = wave * 64 + a * 32 + l31;
      const int i = p0 + a * 32 + l31, q = i < p.total ? i : 0, yy = q / p.W, x = q - yy * p.W, y = yy % p.H;
      uint32_t m = 0x1ff;
      if (y == 0) m &= ~0x007u;
      if (y == p.H - 1) m &= ~0x1c0u;
      if (x == 0) m &= ~0x049u;
      if (x == p.W - 1) m &= ~0x124u;
      in[a] = m;
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
    // operands are fetched two matrix steps ahead, between the matrix instructions
    bf16x8 fa[3][2], fb[3][2];
    uint32_t at[2];                        // of the tap being fetched, step 0
    auto enter = [&](int tap) {
      const int e = p.flip ? 8 - tap : tap, kh = (e * 11) >> 5;         // (e / 3)
      const int shift = kh * p.W + e - 3 * kh;
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const int r = row[a] + shift;
        at[a] = ((in[a] >> e) & 1u) ? (uint32_t)(group * HALO + r * 128 + ((h ^ swizzle128(r)) * 16)) : (uint32_t)ZEROS;
      }
    };
    auto fetch = [&](int set, int x, int s) {
      const int kk = s & 3, tap = s >> 2;
      fa[set][x] = *(const bf16x8*)(area + (at[x] ^ (uint32_t)(kk * 32)));
      fb[set][x] = *(const bf16x8*)(area + (wat[kk] + (uint32_t)(tap * 8192 + x * 4096)));
    };
    enter(0);
    fetch(0, 0, 0); fetch(0, 1, 0);
    fetch(1, 0, 1); fetch(1, 1, 1);
#pragma unroll
    for (int s = 0; s < 36; ++s) {
      const int c = s % 3, n = (s + 2) % 3;
      if (s + 2 < 36 && ((s + 2) & 3) == 0) enter((s + 2) >> 2);
      __builtin_amdgcn_sched_barrier(0);
      acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[c][0], fa[c][0], acc[0][0], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (s + 2 < 36) fetch(n, 0, s + 2);
      __builtin_amdgcn_sched_barrier(0);
      acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[c][1], fa[c][0], acc[0][1], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (s + 2 < 36) fetch(n, 1, s + 2);
      __builtin_amdgcn_sched_barrier(0);
      acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[c][0], fa[c][1], acc[1][0], 0, 0, 0);
      acc[1][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[c][1], fa[c][1], acc[1][1], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // ---- its results: through the wave's patch, so that a store writes whole 128-byte rows; accumulator
  // element 4q + e of a lane: channel 8q + 4h + e, pixel l31
  char* const patch = halo + wave * (PER_WAVE * 1024);
  const uint4 keep = keep8(p.N - j0 - ecol);
  uint4 res[8];
  auto results = [&]() {
    f32x4 bias[2][4];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int q = 0; q < 4; ++q) bias[b][q] = *(const f32x4*)&area[BIAS + (b * 32 + 8 * q + 4 * h) * 4];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          bf16x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float v = acc[a][b][4 * q + e] + bias[b][q][e];
            if (p.relu) v = fmaxf(v, 0.f);
            o[e] = (bf16)v;
          }
          *(bf16x4*)(patch + (a * 32 + l31) * OPITCH + (b * 32 + 8 * q + 4 * h) * 2) = o;
        }
      }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int t = 0; t < 8; ++t) res[t] = *(const uint4*)(patch + (8 * t + erow) * OPITCH + ecol * 2);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      if constexpr (ADD) {
        float v[8], d[8];
        unpack8(res[t], v);
        unpack8(ad[t], d);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += d[e];
        res[t] = pack8(v);
      }
      if constexpr (MASK) {
        res[t] = res[t] & positive8(mk[t]);
      }
      res[t] = res[t] & keep;
    }
  };
  const __amdgpu_buffer_rsrc_t rso = __builtin_amdgcn_make_buffer_rsrc(p.out, 0, p.out_bytes, 0x00020000);
  auto store = [&](int tile) {             // eight instructions always: rows past the batch fail the range check
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const uint32_t i = (uint32_t)(tile * TILE + wave * 64 + 8 * t + erow);
      const u32x4 v = {res[t].x, res[t].y, res[t].z, res[t].w};
      __builtin_amdgcn_raw_buffer_store_b128(v, rso, (int)(i * p.out_pitch + (uint32_t)((j0 + ecol) * 2)), 0, 0);
    }
  };

  if (group < nt) issue_halo(t0 + group);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  // Turn n: group n % 2 computes tile n; the other one finishes tile n - 1 and fetches the halo of n + 1.
#pragma unroll 1
  for (int n = 0; n <= nt; ++n) {
    if ((n & 1) == group) {
      if (n < nt) {
        __builtin_amdgcn_s_setprio(1);
        compute(t0 + n);
        __builtin_amdgcn_s_setprio(0);
      }
    } else if (n > 0) {
      results();
      // (the copies overwrite the patch: its reads have returned; stores go behind the copies, so that
      // waiting for these does not wait for them.  The compiler moves the arithmetic on mask and addend behind the
      // copies and waits for both there, that is, for the copies too; with the builtin wait in front of the copies
      // nothing waits between these and the stores, and 500 models took the same time.)
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (n + 1 < nt) issue_halo(t0 + n + 1);
      asm volatile("" ::: "memory");
      store(t0 + n - 1);
      asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    }
    __syncthreads();
  }
}

}  // namespace

// (Every case of 64 reduction channels that fits: against the gathered-operand product and the halo-tile
// kernel, per iteration of a 4 -> 64 -> 64 -> 64 -> 64 model, 28 x 28 pixels: 2 samples 203 -> 152 us, 64
// samples 259 -> 206, 256 samples 478 -> 371; 32 x 32: 141 -> 127, 207 -> 195, 409 -> 367; 64 -> 200 channels on
// 20 x 33: 138 -> 127, 205 -> 189, 497 -> 454.  Up to 32 outputs the other two waste less.  Weights and halo are laid out
// for exactly 64 channels.  33 to 56 would have to be padded to 64 and stay on the flat run, where they take longer than 64
// do here: 367 x 28 x 28 pixels, 48 -> 48 49 us, 64 -> 48 here 26.)
bool conv_resident_applies(int dtype, const GemmArgs& a) {
  if (dtype != DYNB_BF16 || !a.conv || a.mode == MODE_WGRAD || a.stride != 1) return false;
  if (a.src_w > MAX_W || a.src_w != a.row_w || a.src_h != a.row_h || a.cp != 64 || a.N <= 32) return false;
  if (a.Cf || !a.C || a.M % (a.src_h * a.src_w) || a.lda % 64 || a.ldc % 64 || a.ldb < 576) return false;
  if ((a.mask && a.ldmask % 64) || (a.addend && a.ldadd % 64) || a.ldc < round_up(a.N, 64)) return false;
  // (offsets of 31 bits, with room for the pixels that a halo reaches past the last)
  return ((int64_t)a.M + 512) * a.lda * 2 < (int64_t)1 << 31 && ((int64_t)a.M + 512) * a.ldc * 2 < (int64_t)1 << 31 &&
         (round_up(a.N, 64) + 64) * a.ldb * 2 < (int64_t)1 << 31;
}

int launch_conv_resident(const GemmArgs& a, void* stream) {
  ConvResidentArgs p = {};
  p.src = (const bf16*)a.A; p.pitch = (uint32_t)(a.lda * 2); p.src_bytes = (uint32_t)a.M * p.pitch;
  p.w = (const bf16*)a.B; p.w_pitch = (uint32_t)(a.ldb * 2);
  p.W = a.src_w; p.H = a.src_h; p.total = a.M; p.N = a.N;
  p.tiles = (a.M + TILE - 1) / TILE;
  p.flip = a.conv == 2;
  p.bias = a.mode == MODE_FWD ? a.bias : nullptr;
  p.relu = a.mode == MODE_FWD ? a.relu : 0;
  p.out = (bf16*)a.C; p.out_pitch = (uint32_t)(a.ldc * 2); p.out_bytes = (uint32_t)a.M * p.out_pitch;
  p.mask = a.mode == MODE_DGRAD ? (const bf16*)a.mask : nullptr; p.ldmask = a.ldmask;
  p.addend = a.mode == MODE_DGRAD ? (const bf16*)a.addend : nullptr; p.ldadd = a.ldadd;
  const int blocks_y = (a.N + 63) / 64;
  int bx = 256 / blocks_y;                 // one workgroup per compute unit
  bx = bx < 1 ? 1 : bx > p.tiles ? p.tiles : bx;
  const auto kernel = p.mask ? (p.addend ? conv_resident_kernel<true, true> : conv_resident_kernel<true, false>)
                             : (p.addend ? conv_resident_kernel<false, true> : conv_resident_kernel<false, false>);
  hipLaunchKernelGGL(kernel, dim3(bx, blocks_y), dim3(512), 0, (hipStream_t)stream, p);
  return hipGetLastError() == hipSuccess ? DYNB_OK : fail(DYNB_ERR_HIP, "conv_resident: launch failed");
}

}  // namespace dynb
