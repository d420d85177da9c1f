// Per-worker weight gradient of a 3x3 convolution (NHWC, zero padding 1, stride 1 or 2; bf16),
// straight from the row-major activations:
//   dW_k[kh][kw][ci][co] = sum over worker k's output pixels p of in[src(p, kh, kw)][ci] * dy[p][co]
// The reduction runs over pixels, which are the *rows* of both operands, while an MFMA operand
// wants 8 consecutive reduction indices per lane.  Instead of building transposed copies in
// memory (a patch matrix nine times the activation), tiles are staged in LDS as they lie in
// memory ([pixel][channel]) and fetched with the LDS transpose read of gfx950
// (ds_read_b64_tr_b16): within 16 lanes, lane r supplies the address of 4 channels of pixel
// r/4, and lane l receives channel l of 4 consecutive pixels.
//
// Work split: the rows of a worker are cut into chunks of `chunk_rows` pixels; one workgroup
// takes one chunk, 64 input and 64 output channels, and all nine taps (4 waves: each owns a
// 32 x 32 corner of the 64 x 64 tile for the nine taps, 144 accumulator registers).  A stage is
// 32 pixels x one kernel row (3 taps): 3 x 4 KB of shifted input rows and 4 KB of dy, copied
// global -> LDS asynchronously into a ring of 4 stage buffers.  Chunk results go to a scratch
// area in register order and a second kernel adds the chunks of each worker in a fixed order
// (deterministic, no atomics).  The bias gradient (column sums of dy) rides along as a tenth
// "tap" whose input operand is all ones.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <mutex>
#include <type_traits>

#include "dynb_internal.h"
#include "lds_async.h"

namespace dynb {
namespace {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int S = 4;                         // stage buffers
constexpr int TILE_BYTES = 32 * 128;         // 32 pixels x 64 channels
constexpr int STAGE_BYTES = 4 * TILE_BYTES;  // three shifted input tiles + the dy tile
constexpr int PER = 4;                       // copies per wave and stage
constexpr int SLOTS = 10;                    // nine taps and the column sums of dy
constexpr int TILE_FLOATS = 4 * SLOTS * 16 * 64;   // one chunk result per 64 x 64 channel block:
                                                   // [wave][slot][16 accumulator elements][lane]

__device__ uint4 g_zeros[1];                 // what lanes outside the image or the chunk fetch

__device__ inline void wait_copies(int stages) {   // at most `stages` stages of this wave pending
  switch (stages) {
    case 0: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
    case 1: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PER) : "memory"); break;
    default: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * PER) : "memory"); break;
  }
}

// worker, first row and row count of a chunk
__device__ inline void chunk_span(const Segs& s, const RowChunks& ch, int chunk, int& k, int& r0, int& n) {
  k = 0;
  while (k + 1 < s.K && chunk >= ch.first[k + 1]) ++k;
  r0 = s.off[k] + (chunk - ch.first[k]) * ch.rows;
  n = min(ch.rows, s.off[k + 1] - r0);
}

// Chunk result to memory, in register order: [wave][slot][v/4][lane] x 4 floats.  With two groups of
// four waves the second hands its sums to the first through `red` (TILE_FLOATS floats of LDS).
template <int G>
__device__ inline void store_chunk(f32x16 (&acc)[9], f32x16& colsum, bool sums_columns, int group, int wave,
                                   int lane, f32x4* red, float* out) {
  const int at = wave * SLOTS * 256 + lane;      // in quadruples of floats
  auto quad = [](const f32x16& a, int q) { return f32x4{a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]}; };
  if (G == 2) {
    __syncthreads();                             // the stages are no longer read
    if (group == 1) {
#pragma unroll
      for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) red[at + (t * 4 + q) * 64] = quad(acc[t], q);
#pragma unroll
      for (int q = 0; q < 4; ++q) red[at + (36 + q) * 64] = quad(colsum, q);
    }
    __syncthreads();
    if (group == 1) return;
  }
  f32x4* dst = (f32x4*)out;
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = at + (t * 4 + q) * 64;
      dst[i] = G == 2 ? quad(acc[t], q) + red[i] : quad(acc[t], q);
    }
  if (sums_columns) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = at + (36 + q) * 64;
      dst[i] = G == 2 ? quad(colsum, q) + red[i] : quad(colsum, q);
    }
  }
}

struct ConvWgradArgs {
  const bf16* in; int ldi;           // [samples * H * W][ldi]
  const bf16* dy; int ldd;           // [samples * Ho * Wo][ldd]
  int H, W, Ho, Wo, stride;
  float* partial;                    // [layer][chunk][cin block][cout block][TILE_FLOATS]
  const void* zeros;                 // 16 bytes of zeros in device memory (address of g_zeros: a
                                     // kernel argument stays in scalar registers, the symbol's
                                     // address would be re-loaded around every copy)
};
// Several layers of one geometry in a launch: blockIdx.z = cout block + cobs * layer.  (A type, and kernels, of their own:
// longer arguments and the choice cost launches of one layer 0.5 us.)
struct ConvWgradGroup : ConvWgradArgs {
  int cobs;
  const bf16* more_in[CONV_WGRAD_ITEMS - 1];   // of the layers behind the first
  const bf16* more_dy[CONV_WGRAD_ITEMS - 1];
};

// What a workgroup works on: layer, cout block, the layer's tensors, and the number of its result.
struct Share {
  int cob;
  const bf16 *in, *dy;
  int64_t result;
};
__device__ inline Share share_of(const ConvWgradArgs& p) {
  return {(int)blockIdx.z, p.in, p.dy, (int64_t)(blockIdx.x * gridDim.y + blockIdx.y) * gridDim.z + blockIdx.z};
}
__device__ inline Share share_of(const ConvWgradGroup& p) {
  const int item = (int)blockIdx.z / p.cobs, cob = (int)blockIdx.z - item * p.cobs;
  Share s = {cob, p.in, p.dy, ((int64_t)(item * (int)gridDim.x + (int)blockIdx.x) * (int)gridDim.y + (int)blockIdx.y) * p.cobs + cob};
  // (selected, not indexed: pointers that the compiler finds through a variable index are of no known address
  // space to it, and every store through them a flat one -- 34 -> 55 us)
#pragma unroll
  for (int i = 0; i + 1 < CONV_WGRAD_ITEMS; ++i) {
    s.in = item == i + 1 ? p.more_in[i] : s.in;
    s.dy = item == i + 1 ? p.more_dy[i] : s.dy;
  }
  return s;
}

// G = 2: two groups of four waves take one half of a chunk each, with a ring each, and add their sums
// before they are written.
template <int G, typename Args>
__global__ __launch_bounds__(256 * G) void conv_wgrad_chunk_kernel(Args p, Segs segs, RowChunks ch) {
  __shared__ uint4 ring[G == 1 ? S * STAGE_BYTES / 16 : TILE_FLOATS / 4];
  static_assert(2 * S * STAGE_BYTES <= TILE_FLOATS * 4, "two rings");
  const int group = G == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
  const int lane = threadIdx.x & 63, wave = (threadIdx.x >> 6) & 3;
  const Share share = share_of(p);
  const int chunk = blockIdx.x, cib = blockIdx.y, cob = share.cob;
  int k, r0, n;
  chunk_span(segs, ch, chunk, k, r0, n);
  const int n_blocks = ((n + 31) / 32 + G - 1) / G;   // 32-pixel blocks of a group (the last: maybe fewer)
  r0 += group * n_blocks * 32;
  n -= group * n_blocks * 32;
  n = n < 0 ? 0 : n;
  if (G == 2 && n > n_blocks * 32) n = n_blocks * 32;
  const int T = 3 * ((n + 31) / 32);             // stages of this group

  // ---- global -> LDS: this lane always moves granule (lane & 7) of pixel 8*wave + lane/8 of
  // the block; pixel rows are 128 bytes, and the two 64-byte halves of rows 2,3,6,7,... are
  // swapped so that the transpose reads of 4 neighbouring pixels fall into distinct banks.
  const int prow = 8 * wave + (lane >> 3);
  const int gq = (lane & 7) ^ (((lane >> 4) & 1) << 2);     // logical granule this lane fetches
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)&ring[0] +
                        (uint32_t)(group * S * STAGE_BYTES);
  // output pixel of this lane in the current block: dense row, and (sample, y, x)
  int row = r0 + prow;
  int img = row / (p.Ho * p.Wo), rem = row - img * (p.Ho * p.Wo);
  int oy = rem / p.Wo, ox = rem - oy * p.Wo;
  int left = n - prow;                           // > 0 while this lane's pixel lies in the chunk
  const bf16* in_c = share.in + cib * 64 + gq * 8;
  const bf16* dy_c = share.dy + cob * 64 + gq * 8;
  const bool in_has = cib * 64 + gq * 8 < p.ldi, dy_has = cob * 64 + gq * 8 < p.ldd;   // (narrow rows: no upper half)

  auto issue = [&](int t, int kh) {              // stage t = block t/3, kernel row kh = t%3
    const uint32_t base = lds0 + (uint32_t)((t % S) * STAGE_BYTES + wave * 1024);
    // both candidate addresses are formed unconditionally (coordinates clamped into the image,
    // so always in bounds) and one is selected: no divergent branch around the copy, every
    // stage issues exactly PER copies per wave
    const bool valid = left > 0;
    const int sy = oy * p.stride + kh - 1;
    const bool row_ok = valid && sy >= 0 && sy < p.H;
    const int csy = sy < 0 ? 0 : (sy >= p.H ? p.H - 1 : sy);
    const int line = valid ? (img * p.H + csy) * p.W : 0;      // (pixel indices fit 31 bits)
#pragma unroll
    for (int kw = 0; kw < 3; ++kw) {
      const int sx = ox * p.stride + kw - 1;
      const int csx = sx < 0 ? 0 : (sx >= p.W ? p.W - 1 : sx);
      const bf16* a = in_c + (int64_t)(line + csx) * p.ldi;
      const void* src = (row_ok && in_has && sx >= 0 && sx < p.W) ? (const void*)a : p.zeros;
      async_copy_1k(src, base + kw * TILE_BYTES);
    }
    const bf16* d = dy_c + (int64_t)(valid ? row : 0) * p.ldd;
    const void* src = valid && dy_has ? (const void*)d : p.zeros;
    async_copy_1k(src, base + 3 * TILE_BYTES);
  };
  auto next_block = [&]() {                      // this lane's pixel, 32 pixels on
    row += 32;
    left -= 32;
    ox += 32;
    while (ox >= p.Wo) { ox -= p.Wo; ++oy; }
    while (oy >= p.Ho) { oy -= p.Ho; ++img; }
  };

  // ---- LDS -> MFMA operands.  Wave (wci, wco) owns input channels [32*wci, +32) x output
  // channels [32*wco, +32).  Lane l: group g = l/16 reads pixels 8*(g/2) + r/4 (+4 for the
  // second half of the 8 reduction indices), channels 16*(g%2) + 4*(r%4), r = l%16.
  const int wci = wave & 1, wco = wave >> 1;
  const int g = lane >> 4, r = lane & 15;
  const int fpix = 8 * (g >> 1) + (r >> 2);
  const int fswap = (r >> 3) & 1;                // ((pixel >> 1) & 1) of every pixel this lane reads
  const uint32_t fcol = (uint32_t)((16 * (g & 1) + 4 * (r & 3)) * 2);
  const uint32_t foff_a = (uint32_t)(fpix * 128 + ((wci ^ fswap) * 64)) + fcol;
  const uint32_t foff_b = (uint32_t)(fpix * 128 + ((wco ^ fswap) * 64)) + fcol;
  auto frag = [&](uint32_t tile, uint32_t foff, int kk) {   // 8 reduction indices of k-step kk
    const uint32_t a = tile + foff + (uint32_t)(kk * 16 * 128);
    const s16x4 lo = lds_read_tr(a), hi = lds_read_tr(a + 4 * 128);
    const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  };

  f32x16 acc[9], colsum;
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
#pragma unroll
  for (int v = 0; v < 16; ++v) colsum[v] = 0.f;
  // the waves of the first input-channel block that own input channels [0, 32) also sum dy over
  // the pixels: an MFMA against ones (pixels outside the chunk hold zeros in the dy tile)
  const bool sums_columns = cib == 0 && wci == 0;
  const s16x8 ones_bits = {0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80};
  const bf16x8 ones = __builtin_bit_cast(bf16x8, ones_bits);

  // ---- the stage pipeline: S - 1 stages in flight, one barrier per stage ----
  int issued = 0;                                // stages issued so far (its kernel row = issued % 3)
  auto issue_next = [&]() {
    if (issued < T) {
      const int kh = issued % 3;
      issue(issued, kh);
      if (kh == 2) next_block();
      ++issued;
    }
  };
#pragma unroll
  for (int f = 0; f < S - 1; ++f) issue_next();
  for (int blk = 0; blk < n_blocks; ++blk) {
#pragma unroll
    for (int kh = 0; kh < 3; ++kh) {
      const int t = 3 * blk + kh;
      if (G == 1 || t < T) wait_copies(issued - t - 1);   // stage t of this wave has landed
      __syncthreads();                           // ... of all waves; stage t-1 is no longer read
      if (G == 2 && t >= T) continue;            // (the same for all waves of the group)
      issue_next();                              // into the buffer of stage t-1
      const uint32_t stage = lds0 + (uint32_t)((t % S) * STAGE_BYTES);
      const bf16x8 b0 = frag(stage + 3 * TILE_BYTES, foff_b, 0);
      const bf16x8 b1 = frag(stage + 3 * TILE_BYTES, foff_b, 1);
      if (kh == 1 && sums_columns) {             // once per pixel block
        colsum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b0, ones, colsum, 0, 0, 0);
        colsum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b1, ones, colsum, 0, 0, 0);
      }
#pragma unroll
      for (int kw = 0; kw < 3; ++kw) {
        const bf16x8 a0 = frag(stage + kw * TILE_BYTES, foff_a, 0);
        const bf16x8 a1 = frag(stage + kw * TILE_BYTES, foff_a, 1);
        // first operand = the dimension that is contiguous in the result (output channels)
        acc[kh * 3 + kw] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b0, a0, acc[kh * 3 + kw], 0, 0, 0);
        acc[kh * 3 + kw] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b1, a1, acc[kh * 3 + kw], 0, 0, 0);
      }
    }
  }

  store_chunk<G>(acc, colsum, sums_columns, group, wave, lane, (f32x4*)ring,
                 p.partial + share.result * TILE_FLOATS);
}

// The same for stride 1 on images of 17 to 32 pixels a row: the input rows pass through LDS once.  A stage is
// one input row and one dy row, 32 pixel slots each (zeros beyond the row) with a zero pixel on both sides of
// the input, 8 KB, two copies per wave; ring of ROW_RING stages.  Input row q meets dy rows q - 1, q and
// q + 1 under the kernel rows 2, 1 and 0: the operands of three dy rows stay in registers, so a wave fetches
// 16 operands per row for its 18 matrix instructions instead of 40 (what bounded the version that staged three
// input rows per dy row was the LDS: its reads, 20 KB of copies per row, a barrier for half the work).  The two 16-pixel
// steps of a row are half a stage apart: one is fetched while the other's nine instructions run.
// Combinations outside the worker's rows or across two images are skipped, not multiplied by zeros.
// 512 x 32 x 32 pixels, 64 -> 64 channels: 52 -> 45 us, of which some 8 write the results and 20 are matrix
// instructions; 28 pixels a row took the per-tap kernel: a 64 -> 64 model on 512 x 28 x 28, whole iteration with its
// other convolutions on resident weights, 364 -> 242.
constexpr int ROW_RING = 8;
constexpr int ROW_X = 40 * 128;                  // an input row: eight slots of zeros, 32 pixels; the slots in front of
                                                 // the next stage's row are those behind this one's
constexpr int ROW_DY = ROW_RING * ROW_X + 1024;  // the dy rows, 4 KB each
constexpr int ROW_AREA = ROW_DY + ROW_RING * TILE_BYTES;

template <int G, typename Args>
__device__ __forceinline__ void rows_product(const Args& p, const Segs& segs, const RowChunks& ch, uint4* ring) {
  static_assert(2 * ROW_AREA <= TILE_FLOATS * 4, "two rings in the space of a result");
  const int group = G == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) & 3);
  const Share share = share_of(p);
  const int chunk = blockIdx.x, cib = blockIdx.y, cob = share.cob;
  int k, r0, n;
  chunk_span(segs, ch, chunk, k, r0, n);         // whole image rows
  const int rows = n / p.W, rounds = (rows + G - 1) / G;
  const int T = group == 0 ? rounds : rows - rounds;   // dy rows of this group (the second's: one less if odd)
  const int o0 = r0 / p.W + group * rounds;      // first of them (image * H + y)
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)&ring[0] +
                        (uint32_t)(group * ROW_AREA);
  // the zero slots: never copied into
  for (int e = threadIdx.x & 255; e < (ROW_RING + 1) * 64; e += 256)
    ring[(group * ROW_AREA + (e >> 6) * ROW_X) / 16 + (e & 63)] = make_uint4(0, 0, 0, 0);

  // ---- global -> LDS: wave w copies pixels 8w .. 8w + 7 of both rows; this lane pixel 8w + lane / 8, granule
  // lane % 8 with the halves of slots 2, 3, 6, 7, ... swapped as in the kernel above.  Pixels and channels
  // that do not exist are parked out of the buffer's range (zeros); so is a row in front of the first.
  const int px = 8 * wave + (lane >> 3), gq = (lane & 7) ^ (((lane >> 4) & 1) << 2);
  const i32x4 rsx = buffer_resource(share.in, (uint32_t)segs.off[segs.K] * (uint32_t)p.ldi * 2);
  const i32x4 rsd = buffer_resource(share.dy, (uint32_t)segs.off[segs.K] * (uint32_t)p.ldd * 2);
  const bool x_has = px < p.W && cib * 64 + gq * 8 < p.ldi, dy_has = px < p.W && cob * 64 + gq * 8 < p.ldd;
  uint32_t xoff = x_has ? (uint32_t)((((o0 - 1) * p.W + px) * p.ldi + cib * 64 + gq * 8) * 2) : 0x80000000u;
  uint32_t doff = dy_has ? (uint32_t)(((o0 * p.W + px) * p.ldd + cob * 64 + gq * 8) * 2) : 0x80000000u;
  const uint32_t xstep = (uint32_t)(p.W * p.ldi * 2), dstep = (uint32_t)(p.W * p.ldd * 2);
  uint32_t slot = 0;                             // of the next stage to copy
  auto issue = [&]() {
    async_copy_1k_buffer(rsx, xoff, lds0 + slot * ROW_X + (uint32_t)(1024 + wave * 1024));
    async_copy_1k_buffer(rsd, doff, lds0 + ROW_DY + slot * TILE_BYTES + (uint32_t)(wave * 1024));
    if (x_has) xoff += xstep;
    if (dy_has) doff += dstep;
    slot = slot + 1 == ROW_RING ? 0 : slot + 1;
  };

  // ---- LDS -> MFMA operands (see the kernel above); pixel x under tap kw lies in slot 7 + x + kw
  const int wci = wave & 1, wco = wave >> 1;
  const int g = lane >> 4, r = lane & 15;
  const uint32_t fcol = (uint32_t)((16 * (g & 1) + 4 * (r & 3)) * 2);
  uint32_t foff_a[3];
#pragma unroll
  for (int kw = 0; kw < 3; ++kw) {
    const int hx = 7 + 8 * (g >> 1) + (r >> 2) + kw;
    foff_a[kw] = lds0 + (uint32_t)(hx * 128 + ((wci ^ ((hx >> 1) & 1)) * 64)) + fcol;
  }
  const int fpix = 8 * (g >> 1) + (r >> 2);
  const uint32_t foff_b = lds0 + ROW_DY + (uint32_t)(fpix * 128 + ((wco ^ ((r >> 3) & 1)) * 64)) + fcol;
  // (a row shorter than 32: the slot behind its last dy pixel holds a zero, but under tap 0 it would meet the
  // last input pixel, and 0 x Inf is NaN: that operand comes from a slot of zeros)
  const uint32_t left_lo = 16 + fpix == p.W ? lds0 + fcol : foff_a[0] + 16 * 128;
  const uint32_t left_hi = 20 + fpix == p.W ? lds0 + fcol : foff_a[0] + 20 * 128;
  auto frag = [&](uint32_t a, uint32_t b) {      // 8 reduction indices
    const s16x4 lo = lds_read_tr(a), hi = lds_read_tr(b);
    const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  };

  f32x16 acc[9], colsum;
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
#pragma unroll
  for (int v = 0; v < 16; ++v) colsum[v] = 0.f;
  const bool sums_columns = cib == 0 && wci == 0;
  const s16x8 ones_bits = {0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80};
  const bf16x8 ones = __builtin_bit_cast(bf16x8, ones_bits);

  // Stage t: input row q = o0 - 1 + t, dy row q + 1.  uses: bit kh: dy row q + 1 - kh is this group's and of q's
  // image; bit 3: dy row q + 1 is this group's.
  int iy = o0 % p.H;                             // image row of q + 1
  auto uses_of = [&](int t) {
    const int above = iy;                        // (> 0: q + 1 and q are of one image)
    if (++iy == p.H) iy = 0;                     // image row of q + 2; q's row is iy - 2
    const int q_row = above > 0 ? above - 1 : p.H - 1;
    int u = 0;
    if (t < T) u |= 8 | (above > 0 ? 1 : 0);
    if (t >= 1 && t <= T) u |= 2;
    if (t >= 2 && t <= T + 1 && q_row > 0) u |= 4;
    return u;
  };
  bf16x8 xa[2][3], d[2][3];                      // [step of the row][kw], [step][dy row % 3]
  auto multiply = [&](auto step, auto newest, int uses) {
    constexpr int st = decltype(step)::value, J = decltype(newest)::value;
#pragma unroll
    for (int kh = 0; kh < 3; ++kh) {
      if (!((uses >> kh) & 1)) continue;
#pragma unroll
      for (int kw = 0; kw < 3; ++kw)
        acc[kh * 3 + kw] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(d[st][(J + 3 - kh) % 3], xa[st][kw],
                                                                   acc[kh * 3 + kw], 0, 0, 0);
    }
    if (sums_columns && (uses & 8))
      colsum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(d[st][J], ones, colsum, 0, 0, 0);
  };
  uint32_t at = 0;                               // slot of stage t
  int last_uses = 0;
  auto stage = [&](int t, auto newest) {         // newest: t % 3
    constexpr int J = decltype(newest)::value;
    using Prev = std::integral_constant<int, (J + 2) % 3>;
    // this wave's part of stage t has landed, its reads of stage t - 1 have returned (what they fetched is not
    // used yet, so nothing else waits for them) ...
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * (ROW_RING - 2)) : "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);          // lgkmcnt(0), the other counters at their limits
    __syncthreads();                             // ... and so for every wave
    issue();                                     // into its place
    const uint32_t xs = at * ROW_X, ds = at * TILE_BYTES;
    at = at + 1 == ROW_RING ? 0 : at + 1;
#pragma unroll
    for (int kw = 0; kw < 3; ++kw) xa[0][kw] = frag(foff_a[kw] + xs, foff_a[kw] + xs + 4 * 128);
    d[0][J] = frag(foff_b + ds, foff_b + ds + 4 * 128);
    __builtin_amdgcn_sched_barrier(0);
    multiply(std::integral_constant<int, 1>(), Prev(), last_uses);
    __builtin_amdgcn_sched_barrier(0);
    xa[1][0] = frag(left_lo + xs, left_hi + xs);
#pragma unroll
    for (int kw = 1; kw < 3; ++kw) xa[1][kw] = frag(foff_a[kw] + xs + 16 * 128, foff_a[kw] + xs + 20 * 128);
    d[1][J] = frag(foff_b + ds + 16 * 128, foff_b + ds + 20 * 128);
    __builtin_amdgcn_sched_barrier(0);
    last_uses = uses_of(t);
    multiply(std::integral_constant<int, 0>(), newest, last_uses);
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll 1
  for (int t = 0; t < ROW_RING - 1; ++t) issue();
#pragma unroll
  for (int i = 0; i < 3; ++i) {                  // (registers that a first multiplication may read)
    d[0][i] = d[1][i] = ones;
    xa[0][i] = xa[1][i] = ones;
  }
  // (one stage more for the second step of the last; stages past the end use nothing)
#pragma unroll 1
  for (int t = 0; t < rounds + 3; t += 3) {
    stage(t, std::integral_constant<int, 0>());
    stage(t + 1, std::integral_constant<int, 1>());
    stage(t + 2, std::integral_constant<int, 2>());
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (no copy may land on what follows in this space)

  store_chunk<G>(acc, colsum, sums_columns, group, wave, lane, (f32x4*)ring,
                 p.partial + share.result * TILE_FLOATS);
}

template <int G>
__global__ __launch_bounds__(256 * G, 2) void conv_wgrad_rows_kernel(ConvWgradArgs p, Segs segs, RowChunks ch) {
  __shared__ uint4 ring[G == 1 ? ROW_AREA / 16 : TILE_FLOATS / 4];
  rows_product<G>(p, segs, ch, ring);
}
template <int G>
__global__ __launch_bounds__(256 * G, 2) void conv_wgrad_layers_rows_kernel(ConvWgradGroup p, Segs segs, RowChunks ch) {
  __shared__ uint4 ring[G == 1 ? ROW_AREA / 16 : TILE_FLOATS / 4];
  rows_product<G>(p, segs, ch, ring);
}

// The same for stride 1 and images at least 8 pixels wide: the pixels of all images are one flat run,
// and the three horizontal taps of a kernel row read neighbouring pixels of it, so a stage holds PX
// consecutive output pixels, the three runs of input pixels one image row apart around them (with a
// pixel more on both sides, used through a pixel offset), and nothing is staged per tap.  Rows above
// and below an image are replaced by zeros while they are copied, and so are pixels of other workers
// (zeros in dy alone do not keep an infinity there out of this worker's sums: 0 x Inf is NaN); a run
// also crosses image borders sideways, where the pixel at x = 0 (x = W - 1) must not see the left
// (right) neighbour: for those taps its operand is fetched from a granule of zeros instead.
// CI / CO = 32-channel blocks of the input / output side (1 or 2: up to 32 or 64 channels, not both 2):
// the four waves divide the ten results of a tile -- nine taps and the column sums --
// between them instead of padding the channels to 64.
// A chunk is four to eight stages long, so what bounds a launch is not a rate but the way in and
// out; the code is kept short for that reason too (a wave that runs through code for the first
// time fetches it at about 2 KB per microsecond: with the taps unrolled in every wave, a copy plan
// per copy and the waves' sums combined through LDS, 13 KB, the first figure below was 22).
// 167 x 28 x 28 pixels, 24 -> 24 channels: per-tap kernel 42 us, here 19, 16 with chunks that all run
// at a time (514 workgroups -> 457).
template <int CI, int CO>
struct Flat {
  static constexpr int KS = 4 / (CI * CO);            // waves that share a 32 x 32 channel tile
  static constexpr int ITEMS = (SLOTS + KS - 1) / KS; // results per wave: slots ks, ks + KS, ...
  static constexpr int PX = CI == 2 ? 32 : 64;        // output pixels per stage
  static constexpr int GROUP = 16 / CI;               // pixels per 1 KB copy of an input run, five per run
  static constexpr int IN_ROW = 64 * CI, DY_ROW = 64 * CO;           // bytes per pixel
  static constexpr int IN_TILE = 5 * 1024, DY_COPIES = PX * DY_ROW / 1024;
  static constexpr int STAGE = 3 * IN_TILE + DY_COPIES * 1024;
  static constexpr int RING = 3;                      // stage buffers
  static_assert(IN_TILE >= (PX + 2) * IN_ROW && DY_COPIES <= 8, "copy plan");
};

// Wait until at most n (uniform, <= 6) of this wave's copies are pending.
__device__ inline void wait_at_most(int n) {
  switch (n) {
    case 0: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
    case 1: asm volatile("s_waitcnt vmcnt(1)" ::: "memory"); break;
    case 5: asm volatile("s_waitcnt vmcnt(5)" ::: "memory"); break;
    case 6: asm volatile("s_waitcnt vmcnt(6)" ::: "memory"); break;
    default: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;   // (always safe)
  }
}

template <int CI, int CO, typename Args>
__global__ __launch_bounds__(256, 2) void conv_wgrad_flat_kernel(Args p, Segs segs, RowChunks ch) {
  using F = Flat<CI, CO>;
  __shared__ uint4 ring[F::RING * F::STAGE / 16 + 1];   // (the last granule: zeros)
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const Share share = share_of(p);
  const int chunk = blockIdx.x, cib = blockIdx.y, cob = share.cob;
  int k, r0, n;
  chunk_span(segs, ch, chunk, k, r0, n);
  const int T = (n + F::PX - 1) / F::PX;              // stages
  // the worker's pixels, up to one behind the chunk: what valid taps read
  const int lo = segs.off[k], hi = min(segs.off[k + 1], r0 + n + 1);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)&ring[0];
  const uint32_t lds_zero = lds0 + F::RING * F::STAGE;
  if (threadIdx.x == 0) ring[F::RING * F::STAGE / 16] = make_uint4(0, 0, 0, 0);

  // ---- global -> LDS.  Copy (group q, kh): slots GROUP q .. of input run kh (slot t of a run belongs
  // to output pixel t - 1 of the stage and holds the pixel kh - 1 image rows on).  Waves 0 and 1 copy
  // two groups of the three runs each, wave 2 the fifth group and three of the dy copies, wave 3 the
  // rest of dy.  A lane moves 16 bytes of one pixel.  With 128-byte pixels the two 64-byte halves of
  // pixels 2, 3, 6, 7, ... are swapped (see the kernel above); 64-byte pixels need no swizzle (four
  // neighbouring ones are 256 contiguous bytes).
  const int groups = wave < 2 ? 2 : wave == 2 ? 1 : 0;
  const int dy0 = wave == 3 ? 3 : 0;
  const int dys = wave < 2 ? 0 : wave == 2 ? (F::DY_COPIES < 3 ? F::DY_COPIES : 3)
                                           : (F::DY_COPIES > 3 ? F::DY_COPIES - 3 : 0);
  const int slot0 = 2 * wave * F::GROUP + lane / (4 * CI);       // of this wave's first group
  int pix = r0 + slot0 - 1;                                      // its output pixel (the next group's: + GROUP)
  int x[2], y[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int at = pix + q * F::GROUP < 0 ? 0 : pix + q * F::GROUP;
    const int row = at / p.W;
    x[q] = at - row * p.W;
    y[q] = row % p.H;
  }
  auto granule = [&](int slot, int wide) {
    const int g = lane % (4 * wide);
    return wide == 2 ? g ^ (((slot >> 1) & 1) << 2) : g;         // (slots 8 apart: the same)
  };
  const char* in = (const char*)(share.in + (int64_t)pix * p.ldi + cib * 64 + granule(slot0, CI) * 8);
  const int dslot = dy0 * (16 / CO) + lane / (4 * CO);
  int dpix = r0 + dslot;
  const char* dy = (const char*)(share.dy + (int64_t)dpix * p.ldd + cob * 64 + granule(dslot, CO) * 8);
  const int64_t in_pix = (int64_t)p.ldi * 2, dy_pix = (int64_t)p.ldd * 2;
  const int step_x = F::PX % p.W, step_y = (F::PX / p.W) % p.H;
  auto issue = [&](uint32_t base) {                              // base: LDS address of the stage
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (q >= groups) break;
      const int at = pix + q * F::GROUP;
      const bool live = at >= lo && at < hi;
#pragma unroll
      for (int kh = 0; kh < 3; ++kh) {
        const bool ok = live && (kh != 0 || y[q] > 0) && (kh != 2 || y[q] < p.H - 1);
        const char* src = in + (q * F::GROUP + (kh - 1) * p.W) * in_pix;
        async_copy_1k(ok ? (const void*)src : p.zeros,
                      base + (uint32_t)(kh * F::IN_TILE + (2 * wave + q) * 1024));
      }
      // (the pixel in front of the first is -1: its place was that of pixel 0)
      x[q] += step_x - (at < 0 ? 1 : 0);
      y[q] += step_y;
      if (x[q] < 0) { x[q] += p.W; --y[q]; }
      if (x[q] >= p.W) { x[q] -= p.W; ++y[q]; }
      if (y[q] < 0) y[q] += p.H;
      if (y[q] >= p.H) y[q] -= p.H;
    }
    pix += F::PX;
    in += F::PX * in_pix;
#pragma unroll
    for (int d = 0; d < 5; ++d) {
      if (d >= dys) break;
      const bool ok = dpix + d * (16 / CO) < r0 + n;
      async_copy_1k(ok ? (const void*)(dy + d * (16 / CO) * dy_pix) : p.zeros,
                    base + (uint32_t)(3 * F::IN_TILE + (dy0 + d) * 1024));
    }
    dpix += F::PX;
    dy += F::PX * dy_pix;
  };
  const int copies = 3 * groups + dys;

  // ---- LDS -> MFMA operands (lane layout as in the kernel above)
  const int tile = wave % (CI * CO), wci = tile % CI, wco = tile / CI, ks = wave / (CI * CO);
  const int g = lane >> 4, r = lane & 15;
  auto offset = [&](int hx, int half, int wide) {     // byte offset of this lane's 4 channels of slot hx
    const int w = wide == 2 ? half ^ ((hx >> 1) & 1) : 0;
    return (uint32_t)(hx * 64 * wide + w * 64 + (16 * (g & 1) + 4 * (r & 3)) * 2);
  };
  const int fpix = 8 * (g >> 1) + (r >> 2);
  const uint32_t foff_b = 3 * F::IN_TILE + offset(fpix, wco, CO);
  uint32_t foff_a[F::ITEMS];                          // item i: slot ks + KS i; tap < 9, else column sums
#pragma unroll
  for (int i = 0; i < F::ITEMS; ++i) {
    const int tap = ks + F::KS * i < 9 ? ks + F::KS * i : 0;     // (column sums: fetched, not used)
    foff_a[i] = (tap / 3) * F::IN_TILE + offset(fpix + tap % 3, wci, CI);
  }
  auto frag = [&](uint32_t a0, uint32_t a1) {
    const s16x4 lo = lds_read_tr(a0), hi = lds_read_tr(a1);
    const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  };
  const s16x8 ones_bits = {0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80};
  const bf16x8 ones = __builtin_bit_cast(bf16x8, ones_bits);

  f32x16 acc[F::ITEMS];
#pragma unroll
  for (int i = 0; i < F::ITEMS; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
  int lx = (r0 + fpix) % p.W;                         // x of the first pixel this lane reads in a 16-pixel step
  const int lx_step = 16 % p.W;

#pragma unroll 1
  for (int t = 0; t < 2 && t < T; ++t) issue(lds0 + (uint32_t)(t * F::STAGE));
  uint32_t buf = lds0, nbuf = lds0 + 2 * F::STAGE;    // buffers of stages t and t + 2
  for (int t = 0; t < T; ++t) {
    wait_at_most(t + 1 < T ? copies : 0);             // stage t of this wave has landed
    __syncthreads();                                  // ... of all waves; stage t-1 is no longer read
    if (t + 2 < T) issue(nbuf);
#pragma unroll
    for (int step = 0; step < F::PX / 16; ++step) {
      const uint32_t at_b = buf + step * 16 * F::DY_ROW + foff_b;
      const bf16x8 b = frag(at_b, at_b + 4 * F::DY_ROW);      // (pixels 4 apart: same swizzle)
      // whether the lane's two pixels have a left and a right neighbour
      const int lx4 = lx + 4 >= p.W ? lx + 4 - p.W : lx + 4;
      const bool l0 = lx != 0, l1 = lx4 != 0, q0 = lx != p.W - 1, q1 = lx4 != p.W - 1;
      bf16x8 a[F::ITEMS];
#pragma unroll
      for (int i = 0; i < F::ITEMS; ++i) {
        const int kw = (ks + F::KS * i) % 3;
        const uint32_t at = buf + step * 16 * F::IN_ROW + foff_a[i];
        const bool ok0 = kw == 0 ? l0 : kw == 2 ? q0 : true, ok1 = kw == 0 ? l1 : kw == 2 ? q1 : true;
        a[i] = frag(ok0 ? at : lds_zero, ok1 ? at + 4 * F::IN_ROW : lds_zero);
      }
#pragma unroll
      for (int i = 0; i < F::ITEMS; ++i) {
        if (ks + F::KS * i >= 9) a[i] = ones;
        acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, a[i], acc[i], 0, 0, 0);
      }
      lx += lx_step;
      if (lx >= p.W) lx -= p.W;
    }
    buf = buf == lds0 + 2 * F::STAGE ? lds0 : buf + F::STAGE;
    nbuf = nbuf == lds0 + 2 * F::STAGE ? lds0 : nbuf + F::STAGE;
  }

  float* out = p.partial + share.result * (CI * CO * SLOTS * 1024);
#pragma unroll
  for (int i = 0; i < F::ITEMS; ++i) {
    const int slot = ks + F::KS * i;
    if (slot >= SLOTS || (slot == 9 && (cib != 0 || wci != 0))) continue;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 o = {acc[i][4 * q], acc[i][4 * q + 1], acc[i][4 * q + 2], acc[i][4 * q + 3]};
      *(f32x4*)&out[(((tile * SLOTS + slot) * 4 + q) * 64 + lane) * 4] = o;
    }
  }
}

// dW_k[tap][ci][co] = the chunk results of worker k added in a fixed order, and the bias gradient db_k[co] (slot 9,
// input channel 0).  A tile result of a chunk, 32 x 32 channels, is 4 KB in a row; a workgroup takes PER granules of
// 16 bytes of it, all or a quarter: G groups of PER threads add chunks g, g + G, ... (four independent partial sums, so
// that the loads overlap) and meet in LDS, through which the tile also turns: accumulator element v of lane l belongs to
// output channel 8*(v/4) + 4*(l/32) + v%4 and input channel l%32, and leaves as rows of 128 or 32 bytes.  Whole tiles and
// one group where no worker is many chunks (what counts then are the bytes in flight); 16 groups where one is very many
// and there are few tiles: see conv_wgrad_plan().
// (With 32 quadruples of neighbouring input channels per workgroup, every 16 bytes of a result went to a line of their
// own, and seven of eight threads had nothing to add where a worker is one chunk: 256 -> 256 channels, 15 workers
// of 128 pixels, 85 -> 19 us; 64 -> 64, 8 workers, six layers 25 -> 17; 64 -> 128, 4 workers 10.4 -> 8.7.)
// With MoreResults, several layers: blockIdx.z.
struct NoMore {};
struct MoreResults {
  int chunks;                                  // of a layer
  float* dW[CONV_WGRAD_ITEMS - 1];
  float* db[CONV_WGRAD_ITEMS - 1];
};
template <int G, int PER, typename More>
__global__ __launch_bounds__(G * PER) void conv_wgrad_reduce_kernel(const float* __restrict__ partial,
                                                                    int Cin, int Cout, int ci32, int co32,
                                                                    float* __restrict__ dW,
                                                                    float* __restrict__ db,
                                                                    int64_t group_stride, RowChunks ch, More more) {
  constexpr int PARTS = 256 / PER, WIDE = 32 / PARTS, PITCH = WIDE + 4;   // of a tile; output channels, floats per input channel
  __shared__ f32x4 red[G][32 * PITCH / 4];
  const int k = blockIdx.y, g = threadIdx.x / PER, t = threadIdx.x % PER, lane = t & 63, q = t >> 6;
  const int part = blockIdx.x % PARTS, tile = blockIdx.x / PARTS;
  // slots of the tiles one after the other; of the first input channels' tiles the column sums too
  const int tiles_i = (Cin + 31) / 32;
  const int to = tile / (9 * tiles_i + 1), rest = tile - to * (9 * tiles_i + 1);
  const int slot = rest == 9 * tiles_i ? 9 : rest % 9, ti = rest == 9 * tiles_i ? 0 : rest / 9;
  // (a chunk result: blocks of ci32 x co32 tiles of 32 x 32 channels)
  const int cibs = (tiles_i + ci32 - 1) / ci32, cobs = ((Cout + 31) / 32 + co32 - 1) / co32;
  const int wave = ti % ci32 + ci32 * (to % co32);
  const int64_t tile_floats = (int64_t)ci32 * co32 * SLOTS * 1024, stride = cibs * cobs * tile_floats;
  const float* src = partial + ((int64_t)(ti / ci32) * cobs + to / co32) * tile_floats + (wave * SLOTS + slot) * 1024 + (part * PER + t) * 4;
  if constexpr (std::is_same_v<More, MoreResults>) {
    if (blockIdx.z > 0) {
      src += (int64_t)blockIdx.z * more.chunks * stride;
#pragma unroll
      for (int i = 0; i + 1 < CONV_WGRAD_ITEMS; ++i) {
        dW = (int)blockIdx.z == i + 1 ? more.dW[i] : dW;
        db = (int)blockIdx.z == i + 1 ? more.db[i] : db;
      }
    }
  }
  const int last = ch.first[k + 1];
  f32x4 a0 = {0.f, 0.f, 0.f, 0.f}, a1 = a0, a2 = a0, a3 = a0;
  // (channels that do not exist are not read)
  if (ti * 32 + (lane & 31) < Cin && to * 32 + part * WIDE + 8 * q + 4 * (lane >> 5) < Cout)
    for (int c = ch.first[k] + g; c < last; c += 4 * G) {
      f32x4 v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = *(const f32x4*)(src + min(c + i * G, last - 1) * stride);
      a0 += v[0];
      a1 = c + G < last ? a1 + v[1] : a1;
      a2 = c + 2 * G < last ? a2 + v[2] : a2;
      a3 = c + 3 * G < last ? a3 + v[3] : a3;
    }
  red[g][((lane & 31) * PITCH + 8 * q + 4 * (lane >> 5)) / 4] = (a0 + a1) + (a2 + a3);
  __syncthreads();
#pragma unroll
  for (int e = threadIdx.x; e < 32 * WIDE; e += G * PER) {
    const int cil = e / WIDE, col = e % WIDE, ci = ti * 32 + cil, co = to * 32 + part * WIDE + col;
    if (ci >= Cin || co >= Cout || (slot == 9 && ci > 0)) continue;
    float sum = ((const float*)red[0])[cil * PITCH + col];
#pragma unroll
    for (int i = 1; i < G; ++i) sum += ((const float*)red[i])[cil * PITCH + col];
    float* const dst = slot == 9 ? db + co : dW + ((int64_t)slot * Cin + ci) * Cout + co;
    dst[(int64_t)k * group_stride] = sum;
  }
}

}  // namespace

// address of g_zeros on the current device (looked up once per device)
const void* device_zero_granule() {
  static std::mutex mu;
  static const void* known[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  std::lock_guard<std::mutex> lk(mu);
  if (!known[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(g_zeros)) != hipSuccess) return nullptr;
    known[dev] = p;
  }
  return known[dev];
}

RowChunks make_row_chunks(const Segs& s, int rows) {
  RowChunks ch;
  ch.rows = rows;
  ch.first[0] = 0;
  for (int k = 0; k < s.K; ++k)
    ch.first[k + 1] = ch.first[k] + (s.off[k + 1] - s.off[k] + rows - 1) / rows;
  for (int k = s.K + 1; k <= DYNB_MAX_WORKERS; ++k) ch.first[k] = ch.first[s.K];
  return ch;
}

int conv_wgrad_chunk_rows(int64_t max_rows) {
  // about two chunks per compute unit at the largest batch, whole 32-pixel blocks, and long
  // enough that a chunk's result (147 KB per channel block) is small against what it reads
  int64_t rows = round_up((max_rows + 511) / 512, 32);
  return (int)(rows < 256 ? 256 : rows);
}

int64_t conv_wgrad_scratch_floats(int64_t max_rows, int max_workers, int Cin, int Cout) {
  const int64_t chunks = (max_rows + conv_wgrad_chunk_rows(max_rows) - 1) / conv_wgrad_chunk_rows(max_rows) +
                         max_workers;
  return chunks * ((Cin + 63) / 64) * ((Cout + 63) / 64) * TILE_FLOATS;
}

ConvWgradPlan conv_wgrad_plan(int n, int64_t ldi, int Cin, int H, int W, int64_t ldd, int Cout, int Ho, int Wo, int stride,
                              int chunk_rows, int64_t scratch_floats, const Segs& s) {
  ConvWgradPlan p;
  const int cibs = (Cin + 63) / 64, cobs = (Cout + 63) / 64;
  // Stride 1 on images at least 8 wide (a fragment's eight pixels then hold one border pixel of each
  // kind at most): the flat kernel, whose blocks are only as wide as the channels need.  Whole rows
  // need neither its masks nor its bookkeeping: of 32 pixels with a 64-channel side (3 -> 64
  // channels on 512 x 32 x 32 pixels: 48 us by rows, 57 flat), and of more than 16 (below, the second of the
  // two steps of a row would be empty) with two.  Two sides of more than 32 channels otherwise
  // stay on the per-tap kernel (367 x 28 x 28 pixels, 64 -> 64: 50 us against 54 flat; 24 -> 64: 49 against 36).
  bool by_rows = stride == 1 && W > 16 && W <= 32 && Wo == W && H == Ho && (W == 32 ? Cin > 32 || Cout > 32 : Cin > 32 && Cout > 32);
  by_rows = by_rows && (int64_t)s.off[s.K] * ldi * 2 < (int64_t)1 << 31 && (int64_t)s.off[s.K] * ldd * 2 < (int64_t)1 << 31;
  for (int k = 0; k <= s.K && by_rows; ++k) by_rows = s.off[k] % W == 0;
  const bool flat = stride == 1 && W >= 8 && H == Ho && W == Wo && !by_rows && (Cin <= 32 || Cout <= 32);
  p.kernel = by_rows ? CONV_WGRAD_ROWS : flat ? CONV_WGRAD_FLAT : CONV_WGRAD_TAPS;
  p.ci32 = flat && Cin <= 32 ? 1 : 2;
  p.co32 = flat && Cout <= 32 ? 1 : 2;
  p.ch = make_row_chunks(s, chunk_rows);
  const int own_chunks = p.ch.first[s.K];
  const int64_t per_chunk = (int64_t)cibs * cobs, tile_floats = flat ? (int64_t)p.ci32 * p.co32 * SLOTS * 1024 : TILE_FLOATS;
  // From about two chunks per compute unit on, two chunks are one workgroup's, whose halves meet in LDS:
  // half as many results (147 KB each) to write and to add up.  512 x 32 x 32 pixels, 64 -> 64 channels:
  // 53 + 15.5 us for the product and the sum over chunks -> 51 + 10.3; 512 x 16 x 16, 32 -> 64, stride
  // 2: 31 + 13 -> 30 + 7.  With fewer chunks each has a compute unit to itself, which is worth more.
  p.paired = !flat && n * own_chunks * per_chunk >= 384;
  // Layers of one geometry share a launch, and divide between them the workgroups that one of them would fill the
  // chip with: as many times longer chunks, so that fewer results are written and added up, and one way in and out
  // instead of one each.  64 -> 64 on 512 x 32 x 32, six layers:
  // 6 x (45 + 10) -> 221 + 18 us; 24 -> 24 on 167 x 28 x 28, four: 4 x (16 + 5.5) -> 34 + 6; iterations
  // of 500 residual models of 4 to 300 channels take 0.91 of the time on average, none more than 1.03.
  // Every worker ends with a chunk of its own, so there may be a few chunks more than workgroups that
  // run at a time, which would then run alone at the end: chunks up to a quarter longer (of several layers, whose last
  // chunks are as many times more, up to a half), if that makes them fit.
  const int slots = p.paired ? 256 : 512, step = by_rows ? W : 32;
  const int64_t own = p.paired ? 2 * chunk_rows : chunk_rows;
  int64_t shared = n * (int64_t)s.off[s.K] * per_chunk / slots;
  shared = shared < own ? own : shared > own * n ? own * n : shared;
  const int base = (int)round_up(shared, step);
  const int64_t all = ((int64_t)s.off[s.K] + base - 1) / base * per_chunk * n;
  const int64_t fit = (n > 1 && all <= slots + slots / 8 ? slots : round_up(all, slots)) / per_chunk;
  for (int rows = base; rows <= base + base / (n > 1 ? 2 : 4); rows += step) {
    const RowChunks longer = make_row_chunks(s, rows);
    if ((int64_t)n * longer.first[s.K] > fit && rows > base) continue;
    p.ch = longer;
    if ((int64_t)n * longer.first[s.K] <= fit) break;
  }
  // And as long as it takes for the results of all to fit in the scratch area.  It holds those of one layer at its own
  // chunks, fewer than a chip's worth for small batches (64 -> 64, six layers, iterations of three blocks: 128 images of
  // 16 x 16, two workers, 493 -> 383 us against one launch each; 48 of 32 x 32, five workers, 435 -> 383 against 1 + 2 + 1 + 2
  // layers; 10 % on average over 22 such models, none slower; up to twice as long: the same).
  auto fits = [&](const RowChunks& c) { return (int64_t)n * c.first[s.K] * per_chunk * tile_floats <= scratch_floats; };
  bool together = n == 1 || (int64_t)n * cobs <= 65535;                   // (what a grid takes)
  if (n > 1 && together && !fits(p.ch)) {
    int some = p.ch.rows / step, enough = (int)(own * n * 3 / 2 / step);  // steps per chunk: too few, enough
    p.ch = make_row_chunks(s, enough * step);
    together = enough > some && fits(p.ch);                               // (many workers, each with a last chunk per layer)
    while (together && enough - some > 1) {
      const int half = (some + enough) / 2;
      const RowChunks c = make_row_chunks(s, half * step);
      (fits(c) ? enough : some) = half;
      if (enough == half) p.ch = c;
    }
  }
  if (!together)
    return conv_wgrad_plan((n + 1) / 2, ldi, Cin, H, W, ldd, Cout, Ho, Wo, stride, chunk_rows, scratch_floats, s);
  p.layers = n;
  // The sum over chunks lasts as long as that of the worker with the most of them: one group adds 4 chunks in the
  // time of a read (0.22 us), four groups 16.  Four groups are four times the workgroups, though, 0.003 us per tile and
  // worker, and no faster where one worker's tiles alone keep the memory busy.  With 1, 4 and 16 groups, us:
  // 24 channels, 64 workers, one of them with 32 chunks and the others with one each 4.3, 4.9, 10; 64 of one 6.0, 4.9, 10;
  // 190 of one 13.1, 5.4, 10; 64 channels, 8 workers with 8 each 3.6, 4.5, 7.6; with 24 each 5.6, 5.2, 10.6; 4 workers, 190
  // of one 20, 7.4, 5.4; 256 channels, 8 workers, 48 of one 23, 33, 68; 128 of one 61, 69, 111.
  // (Over 436 such sums the form taken is 0.5 % from the fastest on average and 15 % at most; decided by the mean over
  // the workers, 7 % and a factor of 2.4.  3-24-24 channels on 16 x 16, 700 images of 64 workers, 637 of one: 134 -> 123 us
  // per iteration.)
  int most = 0;
  for (int k = 0; k < s.K; ++k) most = std::max(most, p.ch.first[k + 1] - p.ch.first[k]);
  const int64_t tiles = (int64_t)(9 * ((Cin + 31) / 32) + 1) * ((Cout + 31) / 32) * p.layers;
  p.sum_groups = tiles >= 256 || most <= 4 || most <= tiles * s.K / 16 ? 1 : most > 128 && tiles * s.K < 512 ? 16 : 4;
  return p;
}

int launch_conv_wgrad(const ConvWgradLayer* layers, int n, int64_t ldi, int Cin, int H, int W, int64_t ldd,
                      int Cout, int Ho, int Wo, int stride, int chunk_rows, float* scratch,
                      int64_t scratch_floats, int64_t group_stride, const Segs& s, double flops, double bytes,
                      void* stream) {
  if (Cin <= 0 || Cout <= 0 || n <= 0) return DYNB_OK;
  if (n > CONV_WGRAD_ITEMS) return fail(DYNB_ERR_BADARG, "conv_wgrad: too many layers for one launch");
  const int cibs = (Cin + 63) / 64, cobs = (Cout + 63) / 64;
  uintptr_t addresses = (uintptr_t)scratch;
  for (int i = 0; i < n; ++i) addresses |= (uintptr_t)layers[i].in | (uintptr_t)layers[i].dy;
  if (ldi % 32 || ldd % 32 || ldi < Cin || ldd < Cout || (Cin > 32 && ldi % 64) || (Cout > 32 && ldd % 64) || chunk_rows < 32 || chunk_rows % 32 ||
      (addresses & 15))
    return fail(DYNB_ERR_BADARG, "conv_wgrad: pitches must cover whole 32-channel blocks, 16-byte aligned");
  if (ldi > INT_MAX || ldd > INT_MAX || (int64_t)s.off[s.K] * stride * stride > INT_MAX / 2)
    return fail(DYNB_ERR_UNSUPPORTED, "conv_wgrad: tensor too large for 32-bit pixel indices");
  const void* zeros = device_zero_granule();
  if (!zeros) return fail(DYNB_ERR_HIP, "conv_wgrad: no address for the zero granule");
  if ((int64_t)make_row_chunks(s, chunk_rows).first[s.K] * cibs * cobs * TILE_FLOATS > scratch_floats)
    return fail(DYNB_ERR_BADARG, "conv_wgrad: scratch area too small");
  const ConvWgradPlan plan =
      conv_wgrad_plan(n, ldi, Cin, H, W, ldd, Cout, Ho, Wo, stride, chunk_rows, scratch_floats, s);
  if (plan.layers < n) {
    const double share = (double)plan.layers / n;
    const int rc = launch_conv_wgrad(layers, plan.layers, ldi, Cin, H, W, ldd, Cout, Ho, Wo, stride, chunk_rows, scratch,
                                     scratch_floats, group_stride, s, flops * share, bytes * share, stream);
    return rc ? rc : launch_conv_wgrad(layers + plan.layers, n - plan.layers, ldi, Cin, H, W, ldd, Cout, Ho, Wo, stride,
                                       chunk_rows, scratch, scratch_floats, group_stride, s, flops * (1 - share),
                                       bytes * (1 - share), stream);
  }
  const RowChunks& ch = plan.ch;
  const int nch = ch.first[s.K], ci32 = plan.ci32, co32 = plan.co32;
  const bool paired = plan.paired;
  Timed t(KC_GEMM_WGRAD, stream, flops, bytes);
  ConvWgradGroup a = {};
  MoreResults more = {};
  a.in = (const bf16*)layers[0].in; a.ldi = (int)ldi;
  a.dy = (const bf16*)layers[0].dy; a.ldd = (int)ldd;
  a.H = H; a.W = W; a.Ho = Ho; a.Wo = Wo; a.stride = stride;
  a.partial = scratch; a.zeros = zeros;
  a.cobs = cobs;
  more.chunks = nch;
  for (int i = 1; i < n; ++i) {
    a.more_in[i - 1] = (const bf16*)layers[i].in;
    a.more_dy[i - 1] = (const bf16*)layers[i].dy;
    more.dW[i - 1] = layers[i].dW;
    more.db[i - 1] = layers[i].db;
  }
  const hipStream_t st = (hipStream_t)stream;
  auto launch = [&](auto args) {
    using Args = decltype(args);
    const dim3 grid(nch, cibs, cobs * n), block(paired ? 512 : 256);
    if (plan.kernel == CONV_WGRAD_ROWS) {
      if constexpr (std::is_same_v<Args, ConvWgradGroup>)
        hipLaunchKernelGGL(paired ? conv_wgrad_layers_rows_kernel<2> : conv_wgrad_layers_rows_kernel<1>, grid, block, 0, st, args, s, ch);
      else
        hipLaunchKernelGGL(paired ? conv_wgrad_rows_kernel<2> : conv_wgrad_rows_kernel<1>, grid, block, 0, st, args, s, ch);
    } else if (paired)
      hipLaunchKernelGGL((conv_wgrad_chunk_kernel<2, Args>), grid, block, 0, st, args, s, ch);
    else if (plan.kernel == CONV_WGRAD_TAPS)
      hipLaunchKernelGGL((conv_wgrad_chunk_kernel<1, Args>), grid, block, 0, st, args, s, ch);
    else if (ci32 == 1 && co32 == 1)
      hipLaunchKernelGGL((conv_wgrad_flat_kernel<1, 1, Args>), grid, block, 0, st, args, s, ch);
    else if (ci32 == 1)
      hipLaunchKernelGGL((conv_wgrad_flat_kernel<1, 2, Args>), grid, block, 0, st, args, s, ch);
    else
      hipLaunchKernelGGL((conv_wgrad_flat_kernel<2, 1, Args>), grid, block, 0, st, args, s, ch);
  };
  if (nch > 0) {
    if (n == 1) launch((const ConvWgradArgs&)a);
    else launch(a);
  }
  const unsigned tile_slots = (9 * ((Cin + 31) / 32) + 1) * ((Cout + 31) / 32);
  auto reduce = [&](auto behind) {
    using More = decltype(behind);
    auto as = [&](auto groups, auto granules) {
      constexpr int G = decltype(groups)::value, PER = decltype(granules)::value;
      hipLaunchKernelGGL((conv_wgrad_reduce_kernel<G, PER, More>), dim3(tile_slots * (256 / PER), s.K, n), dim3(G * PER), 0, st,
                         scratch, Cin, Cout, ci32, co32, layers[0].dW, layers[0].db, group_stride, ch, behind);
    };
    if (plan.sum_groups == 1) as(std::integral_constant<int, 1>(), std::integral_constant<int, 256>());
    else if (plan.sum_groups == 4) as(std::integral_constant<int, 4>(), std::integral_constant<int, 64>());
    else as(std::integral_constant<int, 16>(), std::integral_constant<int, 64>());
  };
  if (n == 1) reduce(NoMore());
  else reduce(more);
  return hipGetLastError() == hipSuccess ? DYNB_OK : fail(DYNB_ERR_HIP, "conv_wgrad: launch failed");
}

}  // namespace dynb
