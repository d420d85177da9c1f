// bf16 forward and input-gradient products of dense layers on large tiles: C[i][j] = sum_k A[i][k] B[j][k], both
// operands contiguous in k.
//
// A stage is 64 reduction elements, the whole 128-byte line of every operand row, copied straight into a
// ring of NB stages in LDS (granule g of row r at slot g ^ swizzle128(r)).  What bounds it are three pipes that
// take about as long for a stage of a compute unit -- on 128 x 128 tiles the matrix instructions 512 clocks, the copies
// 740 (23 per kilobyte, whole lines; with half lines, 32-deep stages, 38) and the LDS, fragments and copies
// together, 770 -- and whether they overlap.  A stage is four steps of 16 elements; a step's fragments are fetched one
// step ahead, and fetches and copies stand between the matrix instructions.  The barrier behind a stage's last
// fetch (in front of its last step) releases its buffer, and the copies of stage t + NB follow at once: on 256 x 256
// tiles, whose ring holds only two stages, half of them in that step and half in the next, so that they have two steps
// to land (spread evenly, the last ones arrive late: 4096^3 107 and 122 us); on 128 x 128 tiles, with four stages, evenly.
// 128 x 64 tiles, four waves, where those of 128 x 128 are fewer than half the compute units and 64 x 64 ones more than
// one each (552 clocks of copies per stage and compute unit instead of twice 370; see gemm_small_applies()).
// Eight waves on the larger tiles, two per SIMD: one issues matrix instructions while the other waits for a copy to be accepted.
// Inside the iterations of a 4096-wide model the loop of 4096^3 takes 181 to 201 thousand clocks, of which 131 are matrix work, at
// 1.7 to 1.9 GHz instead of the rated 2.4: 101 - 106 us.  The clock is no constant: in one iteration right after the first ones it
// was 1.2 GHz, and the loop took 158 to 164 thousand clocks and 134 us -- waits for memory get shorter in clocks as these get longer.
//
// Against 32-deep stages in a ring of 160 KB (launches in a row, us): 4096 x 4096 x 4096 forward 122 -> 107, input
// gradient 127 -> 112; 4096 x 4096 x 1024 39 -> 37 and 44 -> 42; 2048^3 25 -> 20 and 26 -> 20; 4096 x 1000 x 4096 41 -> 34;
// 1531 x 2050 x 1024 15.8 -> 11.5 and 18 -> 12.7.  Inside iterations: 2048-2048-2048-256, 2048 rows 28 -> 21 per
// product; 1001-2050-777-101, 1531 rows 17 -> 12; 4096 x 1000 x 4096 59 -> 48; 4096^3 122 - 130 -> 114 - 126.
#include <hip/hip_runtime.h>

#include "device_rows.h"
#include "dynb_internal.h"
#include "gemm_epilogue.h"
#include "lds_async.h"
#include "tile_map.h"

namespace dynb {
namespace {

// SOON: of a stage's copies, eighths that are issued in the last step of the stage that releases its buffer, and in
// the first step of the next; the rest evenly in the steps behind.
template <int BM, int BN, int WM, int WN, int MODE, int NB, int SOON>
__global__ __launch_bounds__(WM * WN * 64) void gemm_lines_kernel(GemmArgs p) {
  constexpr int NW = WM * WN, TM = BM / WM / 32, TN = BN / WN / 32;
  constexpr int CA = BM / 8 / NW, CB = BN / 8 / NW, NC = CA + CB;   // copies per wave and stage: 8 rows each
  constexpr uint32_t STAGE = (BM + BN) * 128;
  static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "whole copies");
  static_assert(NB * STAGE >= NW * 32 * (32 * TN + 4) * 4, "the epilogue's patches fit in the ring");
  __shared__ uint4 ring[NB * STAGE / 16];
  int ti, tj;
  tile_of_block(blockIdx.x, (p.M + BM - 1) / BM, (p.N + BN - 1) / BN, ti, tj);
  const int i0 = ti * BM, j0 = tj * BN;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave % WM, wn = wave / WM, l31 = lane & 31, h = lane >> 5;
  const uint32_t lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)&ring[0];
  // The operands as buffers that begin at the stage's first column and end with the matrix; rows past the edge of a
  // tile repeat the last one (their products are not stored).  Copies past the last stage are issued too, so that the
  // waits stay constants: they read the rows that follow, or zeros, and are never used.
  uint64_t from[2] = {(uint64_t)(uintptr_t)p.A, (uint64_t)(uintptr_t)p.B};
  uint32_t left[2] = {(uint32_t)((int64_t)p.M * p.lda * 2), (uint32_t)((int64_t)p.N * p.ldb * 2)};
  uint32_t off[NC];
#pragma unroll
  for (int u = 0; u < NC; ++u) {
    const bool isA = u < CA;
    const int r = (isA ? CA * wave + u : CB * wave + u - CA) * 8 + (lane >> 3), g = (lane & 7) ^ swizzle128(r);
    const int i = i0 + r < p.M ? i0 + r : p.M - 1, j = j0 + r < p.N ? j0 + r : p.N - 1;
    off[u] = (uint32_t)((isA ? (int64_t)i * p.lda : (int64_t)j * p.ldb) * 2) + g * 16;
  }
  auto copy_one = [&](uint32_t slot, int u) {
    const bool isA = u < CA;
    const i32x4 r = {(int)(uint32_t)from[!isA], (int)(uint32_t)(from[!isA] >> 32), (int)left[!isA], BUFFER_32BIT};
    async_copy_1k_buffer(r, off[u], lds + slot + (isA ? (CA * wave + u) * 1024u : BM * 128u + (CB * wave + u - CA) * 1024u));
  };
  auto next_stage = [&]() {
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      from[o] += 128;
      left[o] = less_128(left[o]);
    }
  };
  f32x16 acc[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
  // copies behind step 3 of the stage before, 0, 1, 2: up to Q[1], Q[2], ...
  constexpr int Q[5] = {0, SOON * NC / 8, 2 * SOON * NC / 8, SOON * NC / 4 + (NC - SOON * NC / 4) / 2, NC};
#pragma unroll 1
  for (int s = 0; s < NB - 1; ++s) {
#pragma unroll
    for (int u = 0; u < NC; ++u) copy_one(s * STAGE, u);
    next_stage();
  }
#pragma unroll
  for (int u = 0; u < Q[1]; ++u) copy_one((NB - 1) * STAGE, u);

  // fragments: lane (l31, h) reads granule 2 kk + h of row l31 of a 32-row block
  const char* const base = (const char*)&ring[0];
  int at[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) at[kk] = (wm * (BM / WM) + l31) * 128 + (((2 * kk + h) ^ swizzle128(l31)) * 16);
  const int to_b = (BM + wn * (BN / WN) - wm * (BM / WM)) * 128;
  bf16x8 fa[2][TM], fb[2][TN];             // [register set: the step's parity]
  auto fetch_one = [&](uint32_t slot, int kk, int f) {
    if (f < TM) fa[kk & 1][f] = *(const bf16x8*)(base + slot + at[kk] + f * 4096);
    else fb[kk & 1][f - TM] = *(const bf16x8*)(base + slot + at[kk] + to_b + (f - TM) * 4096);
  };
  constexpr int NM = TM * TN, NF = TM + TN;
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NB - 2) * NC + Q[1]) : "memory");
  __syncthreads();
#pragma unroll
  for (int f = 0; f < NF; ++f) fetch_one(0, 0, f);
  uint32_t slot = 0, fill = (NB - 1) * STAGE;
#pragma unroll 1
  for (int k = 0; k < p.K; k += 64) {
    const uint32_t next = slot + STAGE == NB * STAGE ? 0 : slot + STAGE;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      if (kk == 3) {
        // this wave's copies of the next stage have landed (behind them, NB - 2 stages) and its reads of this one have
        // returned, and so for every wave
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NB - 2) * NC) : "memory");
        __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0), the other counters at their limits
        __syncthreads();
        next_stage();
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        acc[m % TM][m / TM] =
            __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[kk & 1][m / TM], fa[kk & 1][m % TM], acc[m % TM][m / TM], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        const int first = Q[(kk + 1) & 3], items = NF + Q[((kk + 1) & 3) + 1] - first;
#pragma unroll
        for (int it = m * items / NM; it < (m + 1) * items / NM; ++it) {
          if (it < NF) fetch_one(kk < 3 ? slot : next, (kk + 1) & 3, it);
          else copy_one(kk < 3 ? fill : slot, first + it - NF);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    fill = slot;
    slot = next;
  }
  __builtin_amdgcn_s_waitcnt(0xc07f);      // (fetches past the last stage)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (no copy may land in the patches, or after the LDS has been given back)
  __syncthreads();
  store_product<MODE, TM, TN>(p, p.M, acc, (float*)&ring[0] + wave * 32 * (32 * TN + 4), i0 + wm * (BM / WM),
                              j0 + wn * (BN / WN), [](int i) { return i; });
}

template <int BM, int BN, int WM, int WN, int NB, int SOON>
void launch_as(const GemmArgs& a, hipStream_t st) {
  const dim3 grid(((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN)), block(WM * WN * 64);
  if (a.mode == MODE_FWD)
    hipLaunchKernelGGL((gemm_lines_kernel<BM, BN, WM, WN, MODE_FWD, NB, SOON>), grid, block, 0, st, a);
  else
    hipLaunchKernelGGL((gemm_lines_kernel<BM, BN, WM, WN, MODE_DGRAD, NB, SOON>), grid, block, 0, st, a);
}

}  // namespace

int gemm_lines_tiles(const GemmArgs& a) {
  auto tiles = [&](int m, int n) { return (int64_t)((a.M + m - 1) / m) * ((a.N + n - 1) / n); };
  return tiles(256, 256) >= 192 ? LINES_256 : tiles(128, 128) >= 128 ? LINES_128 : LINES_128X64;
}

int launch_gemm_lines(const GemmArgs& a, void* stream) {
  if (a.mode == MODE_WGRAD || a.conv || a.K % 64 != 0)
    return fail(DYNB_ERR_BADARG, "gemm: products of dense layers take whole 64-deep stages");
  switch (gemm_lines_tiles(a)) {
    case LINES_256: launch_as<256, 256, 2, 4, 2, 4>(a, (hipStream_t)stream); break;
    case LINES_128: launch_as<128, 128, 4, 2, 4, 2>(a, (hipStream_t)stream); break;
    default: launch_as<128, 64, 2, 2, 4, 2>(a, (hipStream_t)stream);
  }
  return hipGetLastError() == hipSuccess ? DYNB_OK : fail(DYNB_ERR_HIP, "gemm launch failed");
}

}  // namespace dynb
