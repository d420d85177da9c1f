// bf16 matrix products with too few 128 x 128 tiles for the 256 compute units, on 64 x 64 tiles: four
// waves of one 32 x 32 matrix-instruction tile each.  Such launches take a few microseconds, so what
// bounds them is the latency of their first loads, the copies into LDS (64 rows of operand per 32
// clocks of matrix work) and, not least, fetching the code itself -- about half a microsecond per
// kilobyte that a wave runs through for the first time.  Hence rolled loops, results stored straight
// from the accumulators, and one path for all edges.  Sums run in the order of the large kernels.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_rows.h"
#include "dynb_internal.h"
#include "lds_async.h"
#include "softmax_head.h"
#include "step_end.h"
#include "tile_map.h"

namespace dynb {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int T = 64;                      // tile side

// Forward and input gradient: C[i][j] = sum_k A[i][k] B[j][k].  A stage is 64 reduction elements, the
// whole 128-byte line of each of the 64 + 64 operand rows (16 copies, four per wave); ring of NB
// stages, all issued ahead of the loop (eight instead of four changed nothing).  A compute unit
// holds one such workgroup, so what bounds a stage is its serial chain: the next stage's operands are on their
// way into the other register set while the matrix instructions of this one run (1024 x 1024 x 3072 17 -> 14 us, 1024 x 10 x 1024 with its loss 8.4
// -> 7.2), and so are the copies, of which a compute unit takes one per 23 clocks: behind the four matrix instructions
// a wave waited for them with nothing left to do.  Addresses are formed behind the last matrix instruction, as a
// vector instruction between two of a chain costs 16 clocks (both: 1024 x 1024 x 1024 7.0 -> 6.7 us, iterations of 600
// models of 4 to 4096 features 1 % faster on average; with the ring unrolled and no address to form, larger models gained
// half a percent more and the smallest lost it to the longer code).  Copies
// past the last stage are still issued (the wait stays a constant); what they read -- the next rows,
// zeros past the matrix -- is never used.
// On 128 x 128 tiles: 1024 x 1024 x 3072 30 us, 1024 x 10 x 1024 14 (without its loss).
constexpr int NB = 4, STAGE = 2 * T * 128;

// With HeadArgs (forward, at most 64 columns) the tile's rows of logits go through the softmax and the loss in
// LDS instead of to memory.
template <int MODE, typename Head>
__global__ __launch_bounds__(256) void gemm_small_kernel(GemmArgs p, Head head) {
  __shared__ uint4 ring[NB * STAGE / 16];
  int ti, tj;
  tile_of_block(blockIdx.x, (p.M + T - 1) / T, (p.N + T - 1) / T, ti, tj);
  const int i0 = ti * T, j0 = tj * T;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l31 = lane & 31, h = lane >> 5, wi = wave & 1, wj = wave >> 1;
  const uint32_t lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)&ring[0];
  // the operands as buffers that begin at the stage's first column and end with the matrix
  uint64_t from[2] = {(uint64_t)(uintptr_t)p.A, (uint64_t)(uintptr_t)p.B};
  uint32_t left[2] = {(uint32_t)((int64_t)p.M * p.lda * 2), (uint32_t)((int64_t)p.N * p.ldb * 2)};
  // copy u of this wave: rows 16 wave + 8 u .. of A (u < 2), of B; rows past the edge repeat the last
  // one (their products are not stored)
  uint32_t off[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int r = 16 * wave + 8 * (u & 1) + (lane >> 3), g = (lane & 7) ^ swizzle128(r);
    const int i = i0 + r < p.M ? i0 + r : p.M - 1, j = j0 + r < p.N ? j0 + r : p.N - 1;
    off[u] = (uint32_t)((u < 2 ? (int64_t)i * p.lda : (int64_t)j * p.ldb) * 2) + g * 16;
  }
  auto copy_one = [&](uint32_t slot, int u) {
    const i32x4 r = {(int)(uint32_t)from[u >> 1], (int)(uint32_t)(from[u >> 1] >> 32), (int)left[u >> 1], BUFFER_32BIT};
    async_copy_1k_buffer(r, off[u], lds + slot + (uint32_t)((u >> 1) * (T * 128) + (2 * wave + (u & 1)) * 1024));
  };
  auto next_stage = [&]() {
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      from[o] += 128;
      left[o] = less_128(left[o]);
    }
  };
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  constexpr bool HEAD = std::is_same_v<Head, HeadArgs>;
  __shared__ int label[HEAD ? T : 1], owned[HEAD ? T : 1];     // of the tile's rows
  int mine = 0;
  if constexpr (HEAD) {
    if (threadIdx.x < T) mine = head.y[min(i0 + (int)threadIdx.x, p.M - 1)];
  }
  // What the epilogue adds to this lane's results (accumulator elements 4q .. 4q+3: row l31, columns 8q + 4h ..)
  // or masks them with, asked for now: fetched where they are used, every value costs a trip to memory.
  const int i = i0 + wi * 32 + l31, ic = i < p.M ? i : p.M - 1;
  float bias[4][4];
  bf16x4 addend[4], mask[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int j = j0 + wj * 32 + 8 * q + 4 * h, jc = j < p.N ? j : 0;   // (rows are padded to 64: whole quads)
    if (MODE == MODE_FWD && p.bias) {
#pragma unroll
      for (int e = 0; e < 4; ++e) bias[q][e] = p.bias[j + e < p.N ? j + e : p.N - 1];
    }
    if (MODE == MODE_DGRAD && p.addend) addend[q] = *(const bf16x4*)((const bf16*)p.addend + (int64_t)ic * p.ldadd + jc);
    if (MODE == MODE_DGRAD && p.mask) mask[q] = *(const bf16x4*)((const bf16*)p.mask + (int64_t)ic * p.ldmask + jc);
  }
#pragma unroll 1
  for (int s = 0; s < NB; ++s) {
#pragma unroll
    for (int u = 0; u < 4; ++u) copy_one((uint32_t)(s * STAGE), u);
    next_stage();
  }
  if constexpr (HEAD) {
    if (threadIdx.x < T) {                 // (while the first copies are on their way)
      owned[threadIdx.x] = rows_of_owner(head.segs, i0 + (int)threadIdx.x);
      label[threadIdx.x] = mine < 0 ? 0 : mine >= p.N ? p.N - 1 : mine;      // keeps the read in bounds
    }
  }
  const int fa = (wi * 32 + l31) * 128, fb = (T + wj * 32 + l31) * 128, sw = swizzle128(l31);
  bf16x8 a[2][4], b[2][4];                 // [register set][step of 16]
  const char *pa[4], *pb[4];               // this lane's operands of the stage that is fetched next
  auto point = [&](uint32_t slot) {
    const char* const base = (const char*)&ring[0] + slot;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const int g = ((2 * kk + h) ^ sw) * 16;
      pa[kk] = base + fa + g;
      pb[kk] = base + fb + g;
    }
  };
  auto fetch_one = [&](int set, int kk) {
    a[set][kk] = *(const bf16x8*)pa[kk];
    b[set][kk] = *(const bf16x8*)pb[kk];
  };
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NB - 1) * 4) : "memory");
  __syncthreads();
  point(0);
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) fetch_one(0, kk);
  uint32_t slot = 0;                       // of the stage whose operands are in, or on their way to, `set`
  point(STAGE);
  auto stage = [&](int set) {
    // this wave's part of the next stage has landed, its reads of this one have returned (its slot takes the
    // next copies) ...
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NB - 2) * 4) : "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);    // lgkmcnt(0), the other counters at their limits
    __syncthreads();                       // ... and so for every wave
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[set][kk], a[set][kk], acc, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      fetch_one(set ^ 1, kk);
      copy_one(slot, kk);
      __builtin_amdgcn_sched_barrier(0);
    }
    next_stage();
    slot = slot + STAGE == NB * STAGE ? 0 : slot + STAGE;
    point(slot + STAGE == NB * STAGE ? 0 : slot + STAGE);
  };
  int k = 0;
#pragma unroll 1
  for (; k + 64 < p.K; k += 128) {
    stage(0);
    stage(1);
  }
  if (k < p.K) stage(0);
  __builtin_amdgcn_s_waitcnt(0xc07f);      // (fetches past the last stage)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (no copy may land after the LDS has been given back)

  if constexpr (HEAD) {
    constexpr int PITCH = T + 4;
    float* const logits = (float*)&ring[0];
    __syncthreads();                       // the last stage is no longer read
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int j = wj * 32 + 8 * q + 4 * h;
      f32x4 v = {acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (p.bias) v[e] += bias[q][e];
        if (p.relu) v[e] = fmaxf(v[e], 0.f);
      }
      *(f32x4*)&logits[(wi * 32 + l31) * PITCH + j] = v;
    }
    __syncthreads();
    // a wave's 16 rows on four lanes each, or on 16 in four rounds
    const int lanes = p.N <= 16 ? 4 : 16, c0 = 4 * (lane & (lanes - 1));
#pragma unroll 1
    for (int r = 16 * wave + lane / lanes; r < 16 * (wave + 1); r += 64 / lanes) {
      const float* const row = logits + r * PITCH;
      const f32x4 z = *(const f32x4*)(row + c0);
      float e[4] = {z[0], z[1], z[2], z[3]};
      const int want = label[r];
      const float loss = softmax_row(lanes, e, c0, p.N, want, row[want], owned[r]);
      if (i0 + r >= p.M) continue;
      bf16* const dz = (bf16*)head.dz + (int64_t)(i0 + r) * head.ldd + c0;
      const bf16x4 o = {(bf16)e[0], (bf16)e[1], (bf16)e[2], (bf16)e[3]}, none = {(bf16)0.f, (bf16)0.f, (bf16)0.f, (bf16)0.f};
      *(bf16x4*)dz = o;
      for (int c = 4 * lanes; c < T; c += 4 * lanes) *(bf16x4*)(dz + c) = none;
      if (c0 == 0) head.rowloss[i0 + r] = loss;
    }
    return;
  }
  if (i >= p.M) return;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int j = j0 + wj * 32 + 8 * q + 4 * h;
    if (j >= p.N) continue;
    const bool whole = j + 3 < p.N;        // (pitches are multiples of 64: aligned)
    f32x4 v = {acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
    bf16* const c = (bf16*)p.C + (int64_t)i * p.ldc + j;
    if (MODE == MODE_FWD) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (p.bias) v[e] += bias[q][e];
        if (p.relu) v[e] = fmaxf(v[e], 0.f);
      }
      if (p.Cf) {
        float* const cf = p.Cf + (int64_t)i * p.ldcf + j;
        if (whole) *(f32x4*)cf = v;
        else
          for (int e = 0; e < 3; ++e)
            if (j + e < p.N) cf[e] = v[e];
      }
    } else {
      if (p.addend) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (float)(bf16)v[e] + (float)addend[q][e];
      }
      if (p.mask) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (!((float)mask[q][e] > 0.f)) v[e] = 0.f;
      }
    }
    if (!p.C) continue;
    const bf16x4 o = {(bf16)v[0], (bf16)v[1], (bf16)v[2], (bf16)v[3]};
    if (whole) *(bf16x4*)c = o;
    else
      for (int e = 0; e < 3; ++e)
        if (j + e < p.N) c[e] = o[e];
  }
}

// Per-worker weight gradient: grads_g[j][i] = sum over worker g's rows of x[row][j] dy[row][i], the bias
// gradient, and with `agg` the weighted average.  A stage is 32 rows of both row-major tensors (8
// copies, two per wave, rows past the worker's last read as zeros); matrix operands come from LDS
// through the transpose read.  A workgroup walks the workers [g0, g1) of its tile; its stages form one
// list, so that the ring never drains between workers.  Results leave as 128-byte runs straight from
// the accumulators.
// Against 128 x 128 tiles: 1024 x 1024, 8 workers, 1024 rows 12 us + 8 (average) -> 17; 3072 x 1024 31
// + 22 -> 24; 2050 x 777, 7 workers, 1531 rows 34 -> 20; 777 x 101 11 + 5 (sum of its parts) + 5
// (biases) -> 7.
// What bounds the stages is the LDS: a wave reads 4 KB through the transpose read for two matrix instructions
// (without stores and copies the three layers of 3072-1024-1024-10 take 19 us, with all 39).  The two 16-row
// steps of a stage are half a stage apart -- one is fetched while the other's product runs -- and four
// workgroups of at most 128 registers a lane share a compute unit instead of three: 41 -> 39 us.
constexpr int WNB = 5, WSTAGE = 2 * 32 * 128;

__device__ inline bf16x8 read_tr(uint32_t a) {   // rows 4 apart: same swizzle
  const s16x4 lo = lds_read_tr(a), hi = lds_read_tr(a + 512);
  const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  return __builtin_bit_cast(bf16x8, v);
}

// One launch serves several layers: their workgroups fill each other's tails (the three layers of
// 3072-1024-1024-10, 8 workers, 1024 rows: 4 + 17 + 24 us in turn -> 39; of 1001-2050-777-101: 7 + 20
// + 27 -> 49).
struct SmallWgrad {
  const void* A; const void* B;                  // dy, x
  int64_t lda, ldb, ldcf;
  int M, N, first, tiles, groups_per_block;      // first: its first workgroup
  float* Cf; float* bias_grad; float* agg; float* bias_agg;
};
struct SmallWgrads {
  SmallWgrad item[WGRAD_SMALL_ITEMS];
  int n;
  int64_t group_stride;
  float lam[DYNB_MAX_WORKERS];
  int ends;                                      // the first workgroups, one per worker, do the step's end
  StepEnd end;
};

// PAST: results, the averages too, leave past the caches (wgrad_small_past below says when).  A kernel of its own
// each: the compiler makes one plain store of the two in a branch.
template <bool PAST>
__global__ __launch_bounds__(256, 4) void wgrad_small_kernel(SmallWgrads grp, Segs segs) {
  __shared__ uint4 ring[WNB * WSTAGE / 16];
  if ((int)blockIdx.x < grp.ends) {
    if (threadIdx.x < 64) end_worker(grp.end, segs, blockIdx.x);
    return;
  }
  const int of_all = (int)blockIdx.x - grp.ends;
  int q = 0;
  while (q + 1 < grp.n && of_all >= grp.item[q + 1].first) ++q;
  const SmallWgrad& p = grp.item[q];
  const int block = of_all - p.first, part = block / p.tiles;
  int ti, tj;
  tile_of_block((uint32_t)(block - part * p.tiles), (p.M + T - 1) / T, (p.N + T - 1) / T, ti, tj);
  const int i0 = ti * T, j0 = tj * T;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l31 = lane & 31, h = lane >> 5, wi = wave & 1, wj = wave >> 1;
  const int g0 = part * p.groups_per_block, g1 = min(g0 + p.groups_per_block, segs.K);
  const uint32_t lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)&ring[0];
  i32x4 rsA = buffer_resource(p.A, 0u), rsB = buffer_resource(p.B, 0u);
  const uint32_t pitchA = (uint32_t)(p.lda * 2), pitchB = (uint32_t)(p.ldb * 2);
  // copy: rows 8 wave .. 8 wave + 7 of a stage; 64-byte halves of rows 2, 3, 6, 7, ... swapped against
  // bank conflicts of the transpose reads; whole 64-feature runs lie within the row pitch
  const int row = 8 * wave + (lane >> 3), gr = (lane & 7) ^ (((row >> 1) & 1) << 2);
  const uint32_t offA = (uint32_t)row * pitchA + (uint32_t)(i0 * 2 + gr * 16);
  const uint32_t offB = (uint32_t)row * pitchB + (uint32_t)(j0 * 2 + gr * 16);
  // next stage to copy: row r of a worker that ends at `end`; a worker without rows has one stage too
  // (all zeros), which writes its zeros like any other result
  int ig = g0, ir = segs.off[g0], iend = segs.off[g0 + 1];
  auto issue = [&](uint32_t slot) {
    rsA[2] = (int)((uint32_t)iend * pitchA);   // (the range check zeroes rows past the worker's last)
    rsB[2] = (int)((uint32_t)iend * pitchB);
    async_copy_1k_buffer(rsA, offA + (uint32_t)ir * pitchA, lds + slot + (uint32_t)(wave * 1024));
    async_copy_1k_buffer(rsB, offB + (uint32_t)ir * pitchB, lds + slot + (uint32_t)(32 * 128 + wave * 1024));
    ir += 32;
    if (ir >= iend && ig < g1) {
      ++ig;                                    // (past the last worker: its zeros again, never used)
      ir = iend;
      iend = ig < g1 ? segs.off[ig + 1] : iend;
    }
  };
  const int tg = lane >> 4, tr = lane & 15;
  auto tr_off = [&](int half) {
    const int rr = 8 * (tg >> 1) + (tr >> 2);
    return (uint32_t)(rr * 128 + (half ^ ((rr >> 1) & 1)) * 64 + (16 * (tg & 1) + 4 * (tr & 3)) * 2);
  };
  const uint32_t ta = lds + tr_off(wi), tb = lds + 32 * 128 + tr_off(wj);
  const bool bias = j0 == 0 && wj == 0;
  const s16x8 ones_bits = {0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80};
  const bf16x8 ones = __builtin_bit_cast(bf16x8, ones_bits);

  f32x16 acc, agg, bsum;
  bf16x8 a[2], b[2];
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = agg[v] = bsum[v] = 0.f;
  float bagg = 0.f;
  // accumulator element v of a lane: row (x feature) 8 (v / 4) + 4h + v % 4, column (dy feature) l31
  const int i = i0 + wi * 32 + l31, jw = j0 + wj * 32 + 4 * h;
  auto store = [&](float* dst, const f32x16& src) {
    if (i >= p.M) return;
    float* d = dst + (int64_t)jw * p.ldcf + i;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int j = 8 * (v / 4) + (v & 3);
      if (jw + j >= p.N) continue;
      float* const e = d + (int64_t)j * p.ldcf;
      if (PAST) __builtin_nontemporal_store(src[v], e);
      else *e = src[v];
    }
  };
#pragma unroll 1
  for (int s = 0; s < WNB - 1; ++s) issue((uint32_t)(s * WSTAGE));
  uint32_t slot = 0, refill = (WNB - 1) * WSTAGE;
#pragma unroll 1
  for (int g = g0; g < g1; ++g) {
    const int rows = segs.off[g + 1] - segs.off[g];
    int r = 0;
    do {
      // (stores count as pending too: the wait then covers more than it has to, never less; the reads of the
      // stage before have returned too, whose second step is not used yet)
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"((WNB - 2) * 2) : "memory");
      __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0), the other counters at their limits
      __syncthreads();                     // the stage of every wave; the one before is no longer read
      issue(refill);
      a[0] = read_tr(ta + slot);
      b[0] = read_tr(tb + slot);
      __builtin_amdgcn_sched_barrier(0);
      if (r > 0) {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[1], a[1], acc, 0, 0, 0);
        if (bias) bsum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, a[1], bsum, 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      a[1] = read_tr(ta + slot + 16 * 128);
      b[1] = read_tr(tb + slot + 16 * 128);
      __builtin_amdgcn_sched_barrier(0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[0], a[0], acc, 0, 0, 0);
      if (bias) bsum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, a[0], bsum, 0, 0, 0);
      refill = slot;
      slot = slot + WSTAGE == WNB * WSTAGE ? 0 : slot + WSTAGE;
      r += 32;
    } while (r < rows);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[1], a[1], acc, 0, 0, 0);
    if (bias) bsum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, a[1], bsum, 0, 0, 0);
    store(p.Cf + (int64_t)g * grp.group_stride, acc);
    if (bias && h == 0 && i < p.M) p.bias_grad[(int64_t)g * grp.group_stride + i] = bsum[0];
    if (p.agg) {
      agg += grp.lam[g] * acc;
      bagg += grp.lam[g] * bsum[0];
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = bsum[v] = 0.f;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (no copy may land after the LDS has been given back)
  if (!p.agg) return;
  store(p.agg, agg);
  if (bias && h == 0 && i < p.M) p.bias_agg[i] = bagg;
}

int64_t tiles64(const GemmArgs& a) { return (int64_t)((a.M + T - 1) / T) * ((a.N + T - 1) / T); }

}  // namespace

static int64_t large_tiles(const GemmArgs& a) { return (int64_t)((a.M + 127) / 128) * ((a.N + 127) / 128); }

// Up to half as many 128 x 128 tiles as compute units (at 204 of them, 1531 x 2050 x 1024, those take
// 12 us and these 20), and where that is more than one of these tiles per compute unit, up to 1024 reduction elements:
// from there on 128 x 64 tiles make up for their longer way in and out with fewer copies (1531 x 777 x 2112 16.3 ->
// 13.6 us; 1531 x 777 x 128 5.6 -> 5.8; 1244 x 1519 x 128 some 2 us more).  Weight gradients, whose larger tiles would have
// to divide the workers or leave the average to another pass, up to the 256 at which the large kernel folds it in.
bool gemm_small_applies(const GemmArgs& a) {
  if (a.conv) return false;
  if (a.mode != MODE_WGRAD) return a.K % 64 == 0 && large_tiles(a) < 128 && (tiles64(a) <= 256 || a.K < 1024);
  return large_tiles(a) < 256;
}

// Parts that the workers of a tile are divided into where the average is left to another pass: until
// the chip is full.
static int worker_parts(const GemmArgs& a, int K) {
  const int64_t parts = 512 / tiles64(a);
  return parts < 1 ? 1 : parts > K ? K : (int)parts;
}

bool wgrad_small_walks(const GemmArgs& a, const Segs& s) { return worker_parts(a, s.K) == 1; }

// Walking all workers takes a workgroup 1 us per worker and 0.18 us per 32 rows.  Folded, and with a pass
// (kernel times): 64 x 10, 64 workers, 512 rows 71 and 7 + 14 us; 512 x 1024, 16 workers, 4096 rows 44
// and 19 + 10; 1024 x 1024, 16 workers, 1024 rows 28 and 18 + 15; 784 x 128, 2 workers, 512 rows 11 and
// 8 + 6.
double wgrad_small_fold_us(const GemmArgs& a, const Segs& s) {
  return fold_us(s.K + 0.0055 * s.off[s.K], worker_parts(a, s.K), (int64_t)a.M * a.N, s.K);
}

// Matrix work is cheaper on 128 x 128 tiles, results are cheaper to leave from 64 x 64 ones, above all
// where rows of the result are no whole lines.  So the large ones take over with enough of them and
// enough rows per worker (kernel times on small and large tiles, 16 workers, at 1024, 4096 and 16384
// rows: 1024 x 1024 18, 29, 75 us and 22, 29, 59; 1024 x 2048 28, 52, 141 and 30, 44, 100; 1500 x 1500
// 71, 64, 211 and 106, 112, 181; 2048 x 256 12, 18, 39 and 13, 19, 37; 768 x 768, whose 36 large tiles
// divide the chip badly, 14, 23, 54 and 22, 27, 56) -- later where these would leave the average to a
// pass and a workgroup of the small ones walks all workers anyway (1024 x 2048, average included: 30,
// 55, 141 and 57, 71, 127).
bool wgrad_small_pays(const GemmArgs& a, const Segs& s, bool average) {
  const int64_t rows = s.off[s.K], large = large_tiles(a);
  if (large < 64) return large != 32 || s.K < 16 || rows < 16384 || rows < 256 * s.K;
  if (average && worker_parts(a, s.K) == 1) return rows < 16384 || rows < 512 * s.K;
  if (a.ldcf % 32) return rows < 8192 || rows * large < (int64_t)131072 * s.K;
  return rows < (s.K < 4 ? 4096 : 2048) || rows * large < (int64_t)16384 * s.K;
}

int launch_gemm_small(const GemmArgs& a, const HeadArgs* head, void* stream) {
  const int64_t tiles = tiles64(a);
  if (tiles >= (int64_t)1 << 31) return fail(DYNB_ERR_UNSUPPORTED, "gemm: too many tiles for one launch");
  const hipStream_t st = (hipStream_t)stream;
  if (head) {
    if (a.mode != MODE_FWD || a.N > T || head->ldd != T || ((uintptr_t)head->dz & 7))
      return fail(DYNB_ERR_BADARG, "gemm: a softmax needs whole rows in one tile");
    hipLaunchKernelGGL((gemm_small_kernel<MODE_FWD, HeadArgs>), dim3((unsigned)tiles), dim3(256), 0, st, a, *head);
  } else if (a.mode == MODE_FWD) {
    hipLaunchKernelGGL((gemm_small_kernel<MODE_FWD, NoHead>), dim3((unsigned)tiles), dim3(256), 0, st, a, NoHead());
  } else if (a.mode == MODE_DGRAD) {
    hipLaunchKernelGGL((gemm_small_kernel<MODE_DGRAD, NoHead>), dim3((unsigned)tiles), dim3(256), 0, st, a, NoHead());
  } else {
    return fail(DYNB_ERR_BADARG, "gemm: weight gradients have a launch of their own");
  }
  return hipGetLastError() == hipSuccess ? DYNB_OK : fail(DYNB_ERR_HIP, "gemm launch failed");
}

// Whether the results of a launch leave past the caches; where its layers differ, by the more weights.
// Rows that are not whole 128-byte lines: through them.  Past them, every piece of a line is written on its own, and what
// the update or a pass reads next is in memory only (1001-2050-777-101, 7 workers, with Adam: 192 -> 182 us; 1000-1000-1000-100,
// 32 workers: 185 -> 120; 2000-1500-20, 8 workers: 109 -> 81).
// Whole lines with the average formed here: past them.  Kept in the L2s, as dirty lines they cost the 3072-1024-1024-10
// model 13 us per iteration at the ends of launches.
// Other whole lines, by the bytes of the launch's results.  Time through the caches over the time past them, whole
// iterations of 1814 models of 32 to 4096 features and 2 to 64 workers, geometric means of the launches of each size:
// below 8 MB 0.99 - 1.00, 8 to 32 MB 1.01 - 1.03 (1.18 at most), 32 to 128 MB 0.99 - 1.03, 128 to 384 MB 0.95 - 0.99,
// from there on 1.00 - 1.04 (1440-1088-1920-32, 64 workers, 349 -> 410 us).  What the update or a pass reads next is then in
// a cache; on the other side, dirty lines that fill the L2s (32 MB) have to go before the launches behind can use
// them, and results that do not fit in the last-level cache (256 MB) displace what these read.
bool wgrad_small_past(const GemmArgs* a, int n, int K) {
  double bytes = 0;
  for (int q = 0; q < n; ++q) bytes += 4.0 * K * a[q].M * a[q].N;
  const bool sized = (bytes >= 8e6 && bytes < 32e6) || bytes >= 384e6;
  int64_t past = 0;
  for (int q = 0; q < n; ++q) {
    const bool lines = !(a[q].ldcf & 31) && !((uintptr_t)a[q].Cf & 127);
    past += (lines && (a[q].agg || sized) ? 1 : -1) * (int64_t)a[q].M * a[q].N;
  }
  return past > 0;
}

int launch_wgrad_small(const GemmArgs* a, int n, const Segs& s, const StepEnd* end, void* stream) {
  if (n > WGRAD_SMALL_ITEMS) return fail(DYNB_ERR_BADARG, "gemm: too many weight gradients for one launch");
  SmallWgrads grp = {};
  double flops = 0, bytes = 0;
  int64_t blocks = 0;
  for (int q = 0; q < n; ++q) {
    const GemmArgs& g = a[q];
    if (g.M <= 0 || g.N <= 0) continue;
    if (!gemm_small_applies(g) || !g.bias_grad || (g.agg && !g.bias_agg) || g.split > 1 ||
        (grp.n && g.group_stride != grp.group_stride))
      return fail(DYNB_ERR_BADARG, "gemm: not a weight gradient of few tiles with its bias gradient");
    if ((g.lda & 7) || (g.ldb & 7) || (((uintptr_t)g.A | (uintptr_t)g.B) & 15))
      return fail(DYNB_ERR_BADARG, "gemm: operands must have 16-byte aligned rows");
    if (s.off[s.K] * g.lda * 2 >= (int64_t)1 << 31 || s.off[s.K] * g.ldb * 2 >= (int64_t)1 << 31)
      return fail(DYNB_ERR_UNSUPPORTED, "gemm: an operand of 2 GiB or more (rows * pitch) is not supported");
    // (the average needs one workgroup to walk all workers of its tile)
    const int64_t tiles = tiles64(g);
    const int parts = g.agg ? 1 : worker_parts(g, s.K), per = (s.K + parts - 1) / parts;
    grp.item[grp.n++] = {g.A, g.B, g.lda, g.ldb, g.ldcf, g.M, g.N, (int)blocks, (int)tiles, per, g.Cf,
                         g.bias_grad, g.agg, g.bias_agg};
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
  Timed t(KC_GEMM_WGRAD_64, stream, flops, bytes);
  const auto kernel = wgrad_small_past(a, n, s.K) ? wgrad_small_kernel<true> : wgrad_small_kernel<false>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)(blocks + grp.ends)), dim3(256), 0, (hipStream_t)stream, grp, s);
  return hipGetLastError() == hipSuccess ? DYNB_OK : fail(DYNB_ERR_HIP, "gemm launch failed");
}

}  // namespace dynb
