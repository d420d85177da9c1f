// Matrix products of the fp32 models on the fp32 matrix instructions (16 x 16 x 4, fp32 products
// and sums).  The models that run in fp32 are small: a product has a few hundred output tiles and
// a reduction of tens to thousands, so what bounds a launch is the length of the serial chain of
// one tile.  16 x 16 tiles have the shortest chain per reduction step (8 clocks; 32 x 32 x 2: 32),
// so every wave takes a tile of its own from end to end, without barriers and without dividing the
// reduction.  An output is one chain of fused multiply-adds in ascending order of the reduction
// index, whatever the tile size -- the same rounding as a plain loop, which keeps the sign of a
// pre-activation next to zero (and with it the ReLU's decision) independent of how the work is split.
// Operands travel global -> LDS asynchronously (a ring of NB blocks private to the wave, NB - 1 in
// flight) and are read from there in the order the matrix instruction wants, four bytes a lane: in
// registers that order costs more vector instructions per block than its four matrix instructions
// take.  Problems with many tiles give each wave 2 x 2 of them (half the copies per instruction).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "dynb_internal.h"
#include "gemm_f32_product.h"
#include "lds_async.h"
#include "step_end.h"
#include "tile_map.h"

namespace dynb {
namespace {

// Per-worker weight gradient, bias gradient and their weighted average in one pass over the
// row-major tensors: grads_g[j][i] = sum over worker g's rows of x[row][j] dy[row][i].  The
// reduction runs over rows; a block is 16 rows of 16 R features per operand, copied as it lies in
// memory (R copies; a row past the worker's last comes from the zero granule), and matrix instruction t
// reads row 4t + kg: no transposed copies.  A wave walks workers of its tile in ascending order, blocks
// in flight across worker boundaries: all of them where it forms the average too (the lane that stores
// an element keeps its weighted sum), else a share.  The waves of the first tile column sum dy
// alongside: the bias gradient.
// 3072 x 512 weights, 4 workers, 256 rows: 25 us + 5 (bias) + 6 (average) + 10 (transposed
// copies) -> 25 us; 785 x 301, 7 workers, 785 rows: 28 + 5 + 4 + 12 -> 19 us.
// One launch serves every layer of a model (a launch is bound by the chain of a wave, hardly by any
// rate, so the waves of one layer hide those of another; 785-301-97-10: 19 + 17 + 17 us for the three
// layers one after the other -> 25 together, 3072-512-512-10: 24 + 10 + 9 -> 36).
// What stretches that chain is not the memory (rings twice as deep: the same) but what a wave that has its SIMD
// for itself issues between the matrix instructions: a vector instruction as in gemm_f32_product.h, and a taken
// branch some 60 clocks.  So a step has one vector instruction and no branch that is taken: operands are buffers
// that end with the worker's rows, so that no lane compares and selects; the tiles that sum the bias
// gradient are a variant of their own; and what ends a worker stands behind the loop over its blocks, once.  134
// tiles, 785 rows of one worker: 380 -> 250 clocks per 16 rows.  785-301-97-10, 7 workers, all layers: 24.6 -> 18 us;
// 3072-512-512-10, 4 workers (2 x 2 tiles, 30 MB of results): 28.7 -> 21.5.
enum { TILE_1, TILE_2, TILE_1_LONG };
struct WgradItem {
  const void* A; const void* B;            // dy, x
  int64_t lda, ldb, ldcf;
  int M, N, first, kind;                   // first: its first workgroup; kind: TILE_1 ..
  int tiles, per;                          // workgroups tiles * part .. take workers per * part ..
  float* Cf; float* bias_grad; float* agg; float* bias_agg;
};
struct WgradGroup {
  WgradItem item[WGRAD_F32_ITEMS];
  int n;
  int64_t group_stride;
  const void* zeros;
  float lam[DYNB_MAX_WORKERS];
  int ends;                                // the first workgroups, one per worker, do the step's end
  StepEnd end;
};
// (20 KB: eight waves on a compute unit, two per SIMD.  24 left room for six, and launches of many waves
// went in uneven rounds: 1024 x 1024, 4096 rows, one worker 150 -> 95 us)
constexpr uint32_t WGRAD_RING = 20 * KB;

// Granule g of a block's row r sits at slot g ^ swizzle(r): the four rows that a matrix instruction
// reads 16 features of then take all 64 banks.
template <int R>
__device__ inline int swizzle(int r) { return R == 1 ? 0 : 4 * ((r >> 1) & 1); }

// LONG: rows whose offsets within a block or a tile do not fit 32 bits.  Blocks are then copied by address, like the
// first one of every wave.
template <int R, bool BIAS, bool LONG = false>
__device__ __forceinline__ void wgrad_f32_tile(const WgradItem& item, const WgradGroup& grp, const Segs& segs,
                                               int part, int ti, int tj, uint4* ring_area) {
  constexpr int NB = R == 1 ? 10 : 5, S = 16 * R, C = 2 * R;   // copies per block: R of dy, R of x
  constexpr uint32_t SLOT = C * KB;
  using Offset = std::conditional_t<LONG, uint64_t, uint32_t>;
  static_assert(NB * SLOT == WGRAD_RING, "ring");
  const WgradItem p = item;
  const int lane = threadIdx.x, l15 = lane & 15, kg = lane >> 4;
  const int i0 = ti * S, j0 = tj * S;
  const int g0 = part * p.per, g1 = min(g0 + p.per, segs.K);
  const uint32_t lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)&ring_area[0];

  // Every worker has at least one block, so that an idle worker's zeros are written like any other result.
  // (The workers' row counts and weights sit in a register, one worker per lane: a scalar load
  // would make every wait for the operand fetches wait for it too.)
  const int rowsv = segs.off[lane + 1] - segs.off[lane];
  const float lamv = grp.lam[lane];
  auto rows_of = [&](int g) { return __builtin_amdgcn_readlane(rowsv, g); };
  // copy c < R: rows (16 / R) c .. of dy, else of x.  This lane's 16 bytes of a block, from the block's first
  // row (16 R features from a multiple of 16 R on lie within the row pitch).  Each operand is a buffer that begins
  // there and ends with the worker's rows, or the block: what lies behind reads as zeros.
  constexpr int LPR = 4 * R;               // lanes per row
  const int lrow = lane / LPR;
  const Offset pitch[2] = {(Offset)p.lda * 4, (Offset)p.ldb * 4};   // (16 rows below 2^31 bytes: see launch_wgrad_f32())
  uint64_t base[2] = {(uint64_t)(uintptr_t)((const float*)p.A + segs.off[g0] * p.lda + i0),
                      (uint64_t)(uintptr_t)((const float*)p.B + segs.off[g0] * p.ldb + j0)};
  Offset off[C];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int row = lrow + (16 / R) * (c % R), g = (lane & (LPR - 1)) ^ swizzle<R>(row);
    off[c] = row * pitch[c / R] + 16 * g;
  }
  // Copies the next block; rows past the worker's last, and blocks past the last worker, are zeros.
  int copied = g0, to_copy = segs.off[g0 + 1] - segs.off[g0];   // worker, its rows from this block on
  const int first_rows = to_copy;
  auto issue = [&](uint32_t slot, auto by_address) {
    const uint32_t rows = to_copy < 16 ? to_copy : 16;
#pragma unroll
    for (int o = 0; o < 2; ++o) {
#pragma unroll
      for (int c = 0; c < R; ++c) {
        const uint32_t to = lds + slot + (o * R + c) * KB;
        if constexpr (by_address) {
          const bool in = lrow + (16 / R) * c < (int)rows;
          async_copy_1k(in ? (const void*)(uintptr_t)(base[o] + off[o * R + c]) : grp.zeros, to);
        } else {
          const i32x4 r = {(int)(uint32_t)base[o], (int)(uint32_t)(base[o] >> 32), (int)(rows * pitch[o]), BUFFER_32BIT};
          async_copy_1k_buffer(r, off[o * R + c], to);
        }
      }
      base[o] += rows * pitch[o];
    }
    to_copy -= 16;
    if (__builtin_expect(to_copy <= 0, 0)) to_copy = ++copied < g1 ? rows_of(copied) : 0;
  };
  constexpr std::bool_constant<LONG> other_blocks = {};
  float f[2][C][4];                        // [register set][16 features of dy / x][matrix instruction]
  const char* const ring = (const char*)&ring_area[0];
  uint32_t at[R];
#pragma unroll
  for (int u = 0; u < R; ++u)              // (row 4t + kg: its swizzle does not depend on t)
    at[u] = 64 * R * kg + ((64 * u) ^ (16 * swizzle<R>(kg))) + 4 * l15;
  auto fetch_one = [&](int set, uint32_t slot, int t) {
#pragma unroll
    for (int u = 0; u < R; ++u) {
      const char* const a = ring + (slot + at[u]) + t * (256 * R);
      f[set][u][t] = *(const float*)a;
      f[set][R + u][t] = *(const float*)(a + R * KB);
    }
  };
  f32x4 acc[R][R], agg[R][R];              // [x block][dy block]
  float bsum[R], bagg[R];
#pragma unroll
  for (int u = 0; u < R; ++u) {
    bsum[u] = bagg[u] = 0.f;
#pragma unroll
    for (int w = 0; w < R; ++w) acc[u][w] = agg[u][w] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // accumulator element v of a lane: row (x feature) 4 * kg + v, column (dy feature) l15
  const bool in_row = i0 + l15 < p.M, in_row2 = i0 + 16 + l15 < p.M;
  auto store = [&](float* out, const f32x4 (&v)[R][R]) {
#pragma unroll
    for (int u = 0; u < R; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = 16 * u + 4 * kg + e;
        const Offset o = (Offset)j * (Offset)p.ldcf + l15;
        if (j0 + j < p.N) {
          if (in_row) out[o] = v[u][0][e];
          if (R > 1 && in_row2) out[o + 16] = v[u][R - 1][e];
        }
      }
  };

  issue(0, std::true_type());
#pragma unroll 1
  for (uint32_t s = SLOT; s < NB * SLOT; s += SLOT) issue(s, other_blocks);
  wait_pending<(NB - 1) * C>();
#pragma unroll
  for (int t = 0; t < 4; ++t) fetch_one(0, 0, t);
  // (a block past the last is zeros and belongs to no worker.  Stores count as pending too: the
  // wait then covers more than it has to, never less)
  uint32_t slot = 0;
  auto step = [&](int set) {
    const uint32_t ahead = slot + SLOT == NB * SLOT ? 0 : slot + SLOT;
    wait_pending<(NB - 2) * C>();
#pragma unroll
    for (int t = 0; t < 4; ++t) {
#pragma unroll
      for (int w = 0; w < R; ++w)
#pragma unroll
        for (int u = 0; u < R; ++u)
          acc[u][w] = __builtin_amdgcn_mfma_f32_16x16x4f32(f[set][R + u][t], f[set][w][t], acc[u][w], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (t == 0) wait_reads();            // (of `slot`, before it is copied into)
      if (t < 2) {
        fetch_one(set ^ 1, ahead, 2 * t);
        fetch_one(set ^ 1, ahead, 2 * t + 1);
      } else if (t == 2) {
        issue(slot, other_blocks);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (BIAS) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int w = 0; w < R; ++w) bsum[w] += f[set][w][t];
    }
    slot = ahead;
  };
  int g = g0, left = first_rows;
  float* out = p.Cf + (int64_t)g0 * grp.group_stride + (int64_t)j0 * p.ldcf + i0;
#pragma unroll 1
  for (;;) {
#pragma unroll 1
    for (;;) {
      step(0);
      left -= 16;
      if (left <= 0) {                     // (an odd number of blocks: the next one's operands into the first set)
        wait_reads();
#pragma unroll
        for (int t = 0; t < 4; ++t) fetch_one(0, slot, t);
        break;
      }
      step(1);
      left -= 16;
      if (left <= 0) break;
    }
    // ---- end of worker g ----
    const float lam = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(lamv), g));
    store(out, acc);
#pragma unroll
    for (int u = 0; u < R; ++u)
#pragma unroll
      for (int w = 0; w < R; ++w) {
        agg[u][w] += lam * acc[u][w];
        acc[u][w] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    if (BIAS) {
#pragma unroll
      for (int w = 0; w < R; ++w) {
        float v = bsum[w];
        v += __shfl_xor(v, 16);
        v += __shfl_xor(v, 32);
        bagg[w] += lam * v;
        bsum[w] = 0.f;
        const int i = i0 + 16 * w + l15;
        if (kg == 0 && i < p.M) p.bias_grad[(int64_t)g * grp.group_stride + i] = v;
      }
    }
    if (++g >= g1) break;
    left = rows_of(g);
    out += grp.group_stride;
  }
  wait_pending<0>();                       // (no copy may land after the LDS has been given back)
  if (!p.agg) return;
  store(p.agg + (int64_t)j0 * p.ldcf + i0, agg);
  if (BIAS && kg == 0) {
#pragma unroll
    for (int w = 0; w < R; ++w)
      if (i0 + 16 * w + l15 < p.M) p.bias_agg[i0 + 16 * w + l15] = bagg[w];
  }
}

__global__ __launch_bounds__(64) void wgrad_f32_kernel(WgradGroup grp, Segs segs) {
  __shared__ uint4 ring_area[WGRAD_RING / 16];
  const int block = (int)blockIdx.x - grp.ends;
  if (block < 0) {
    end_worker(grp.end, segs, blockIdx.x);
    return;
  }
  int q = 0;
  while (q + 1 < grp.n && block >= grp.item[q + 1].first) ++q;
  const WgradItem& p = grp.item[q];
  const int S = p.kind == TILE_2 ? 32 : 16, part = (block - p.first) / p.tiles;
  int ti, tj;
  tile_of_block(block - p.first - part * p.tiles, (p.M + S - 1) / S, (p.N + S - 1) / S, ti, tj);
  if (p.kind == TILE_2 && tj == 0) wgrad_f32_tile<2, true>(p, grp, segs, part, ti, tj, ring_area);
  else if (p.kind == TILE_2) wgrad_f32_tile<2, false>(p, grp, segs, part, ti, tj, ring_area);
  else if (p.kind == TILE_1 && tj == 0) wgrad_f32_tile<1, true>(p, grp, segs, part, ti, tj, ring_area);
  else if (p.kind == TILE_1) wgrad_f32_tile<1, false>(p, grp, segs, part, ti, tj, ring_area);
  else if (tj == 0) wgrad_f32_tile<1, true, true>(p, grp, segs, part, ti, tj, ring_area);
  else wgrad_f32_tile<1, false, true>(p, grp, segs, part, ti, tj, ring_area);
}

template <int R>
void launch_as(const GemmArgs& a, unsigned blocks, hipStream_t st) {
  const dim3 grid(blocks), block(64);
  if (a.mode == MODE_FWD)
    hipLaunchKernelGGL((gemm_f32_kernel<MODE_FWD, R, NoHead>), grid, block, 0, st, a, NoHead());
  else
    hipLaunchKernelGGL((gemm_f32_kernel<MODE_DGRAD, R, NoHead>), grid, block, 0, st, a, NoHead());
}

}  // namespace

// 2 x 2 tiles per wave once that gives each of the chip's 1024 SIMDs a wave: below that the chain
// of one wave, four times as long, outweighs the halved copies.
static int64_t tiles_with(const GemmArgs& a, int side) {
  return (int64_t)((a.M + side - 1) / side) * ((a.N + side - 1) / side);
}
static int tile_side(const GemmArgs& a) { return tiles_with(a, 32) >= 1024 ? 32 : 16; }

// For a weight gradient the workers count too: they are divided over waves (512 x 512, 16 workers, 16384
// rows: 186 us in single tiles, 80 in 2 x 2; three such layers, 8 workers, 65536 rows, whose operands no longer stay in the
// caches, forward and backward 7060 and 3430; 4 workers and 1024 rows, at the line, 15 and 16.  The line is older than the
// chain without vector instructions: two layers of 256 x 256, 8 workers, 1024 rows, on its other side, 14 and 10.5).
static int wgrad_side(const GemmArgs& a, const Segs& s) { return tiles_with(a, 32) * s.K >= 1024 ? 32 : 16; }

// Workers per wave of a weight gradient that leaves the average to another pass: eight waves of this ring
// fit on a compute unit (64 x 10, 16 workers: 512 rows 14.5 -> 7 us, 4096 rows 43 -> 8.3, 16384 rows 139 ->
// 14.5 against one wave per tile; 512 x 512, 8 workers, 1024 rows 32 -> 13).
static int workers_per_wave(const GemmArgs& a, int K, int side) {
  const int64_t shares = 2048 / tiles_with(a, side);
  return shares < 1 ? K : shares > K ? 1 : (K + (int)shares - 1) / (int)shares;
}
bool wgrad_f32_walks(const GemmArgs& a, const Segs& s) { return workers_per_wave(a, s.K, wgrad_side(a, s)) == s.K; }
// The rule counts 0.06 us per 16 rows and 0.7 us per worker of a wave of 16 x 16 tiles, fitted over whole iterations
// before the chain lost its vector instructions (now a wave that has its SIMD for itself takes 0.11 and 0.55).  Where 2 x 2
// tiles of divided workers fill the chip instead, they are worth a pass of 5 us from 1700 rows times 1024 small tiles on.
// Weight gradients folded, and without the pass; in brackets with it, per iteration: 512 x 512, 8 workers, 1024 rows 20 and
// 14.5 us (33.2, 34.0), 1536 26 and 16 (44.9, 41.8), 4096 50 and 26 (87, 69); 576 x 576, 1024 rows 21.5 and 17.2 (40.3, 42.3),
// 16384 rows 234 and 146 (390, 318); 785-301-97-10, 7 workers 18.6 and 15 (47.9, 52.4).  Of 21 models the rule
// takes the faster side of 20; two layers of 256 x 256, 8 workers, 1024 rows would be faster folded (35 us, 41).
double wgrad_f32_fold_us(const GemmArgs& a, const Segs& s) {
  if (wgrad_side(a, s) != tile_side(a) && tiles_with(a, 16) * s.off[s.K] > 1700 * 1024) return 1e30;
  const int per = workers_per_wave(a, s.K, tile_side(a));
  return fold_us(0.7 * s.K + 0.0036 * s.off[s.K], (s.K + per - 1) / per, (int64_t)a.M * a.N, s.K);
}

// Single tiles keep the byte offset of a lane from their first row in 32 bits.
static int product_side(const GemmArgs& a) {
  const int64_t pitch = a.lda > a.ldb ? a.lda : a.ldb;
  return 16 * 4 * pitch < (int64_t)1 << 32 ? tile_side(a) : 32;
}

// (a tile holds whole rows)
bool gemm_f32_head_applies(const GemmArgs& a) { return a.mode == MODE_FWD && a.N <= 16 && product_side(a) == 16; }

int launch_gemm_f32(const GemmArgs& a, const HeadArgs* head, void* stream) {
  if (a.mode == MODE_WGRAD || a.K % 64 != 0)
    return fail(DYNB_ERR_BADARG, "gemm: fp32 products take whole pairs of 32-deep blocks");
  const int side = product_side(a);
  const int64_t n = tiles_with(a, side);
  if (n >= (int64_t)1 << 31) return fail(DYNB_ERR_UNSUPPORTED, "gemm: too many tiles for one launch");
  if (head) {
    if (!gemm_f32_head_applies(a) || head->ldd != COL_PAD || ((uintptr_t)head->dz & 15))
      return fail(DYNB_ERR_BADARG, "gemm: a softmax needs whole rows in one tile");
    launch_gemm_f32_head(a, *head, (unsigned)n, stream);
  } else if (side == 32) launch_as<2>(a, (unsigned)n, (hipStream_t)stream);
  else launch_as<1>(a, (unsigned)n, (hipStream_t)stream);
  return hipGetLastError() == hipSuccess ? DYNB_OK : fail(DYNB_ERR_HIP, "gemm launch failed");
}

// Offsets within a block of 16 rows, and within the 32 rows of a tile of the result, are 32-bit in the tiles that copy
// through buffers.
static bool wgrad_rows_long(const GemmArgs& g) {
  return 16 * 4 * std::max(g.lda, g.ldb) >= (int64_t)1 << 31 || 32 * 4 * g.ldcf >= (int64_t)1 << 31;
}

int launch_wgrad_f32(const GemmArgs* a, int n, const Segs& s, const StepEnd* end, void* stream) {
  if (n > WGRAD_F32_ITEMS) return fail(DYNB_ERR_BADARG, "gemm: too many weight gradients for one launch");
  WgradGroup grp = {};
  grp.zeros = device_zero_granule();
  if (!grp.zeros) return fail(DYNB_ERR_HIP, "gemm: no address for the zero granule");
  double flops = 0, bytes = 0;
  int64_t blocks = 0, wide = 0;
  for (int q = 0; q < n; ++q) wide += tiles_with(a[q], 32);
  for (int q = 0; q < n; ++q) {
    const GemmArgs& g = a[q];
    if (g.M <= 0 || g.N <= 0) continue;
    if (g.mode != MODE_WGRAD || !g.bias_grad || (g.agg && !g.bias_agg) ||
        (grp.n && g.group_stride != grp.group_stride))
      return fail(DYNB_ERR_BADARG, "gemm: an fp32 weight gradient writes the bias gradient too");
    if ((g.lda & 3) || (g.ldb & 3) || (((uintptr_t)g.A | (uintptr_t)g.B) & 15))
      return fail(DYNB_ERR_BADARG, "gemm: operands must have 16-byte aligned rows");
    // (a wave that folds the average in walks all workers: then the tiles alone have to fill the chip,
    // those of all layers together -- three of 512 x 512, 8 workers, 1024 rows: 35 us, and 41 with 2 x 2 tiles)
    const bool long_rows = wgrad_rows_long(g);
    const int side = long_rows || (g.agg && wide < 1024) ? 16 : wgrad_side(g, s);
    const int64_t tiles = tiles_with(g, side);
    const int per = g.agg ? s.K : workers_per_wave(g, s.K, side);
    if (blocks + tiles * ((s.K + per - 1) / per) >= (int64_t)1 << 31)
      return fail(DYNB_ERR_UNSUPPORTED, "gemm: too many tiles for one launch");
    grp.item[grp.n++] = {g.A, g.B, g.lda, g.ldb, g.ldcf, g.M, g.N, (int)blocks,
                         long_rows ? TILE_1_LONG : side == 32 ? TILE_2 : TILE_1, (int)tiles,
                         per, g.Cf, g.bias_grad, g.agg, g.bias_agg};
    grp.group_stride = g.group_stride;
    if (g.agg)
      for (int k = 0; k < s.K; ++k) grp.lam[k] = g.lam[k];   // (of the call: the same for every layer)
    blocks += tiles * ((s.K + per - 1) / per);
    flops += g.alg_flops;
    bytes += g.alg_bytes;
  }
  if (end) {
    grp.ends = s.K;
    grp.end = *end;
  }
  if (!grp.n && !grp.ends) return DYNB_OK;
  Timed t(KC_GEMM_WGRAD, stream, flops, bytes);
  hipLaunchKernelGGL(wgrad_f32_kernel, dim3((unsigned)(blocks + grp.ends)), dim3(64), 0, (hipStream_t)stream, grp, s);
  return hipGetLastError() == hipSuccess ? DYNB_OK : fail(DYNB_ERR_HIP, "gemm launch failed");
}

}  // namespace dynb
