// The kernel of the fp32 forward and input-gradient products, shared by the plain ones (gemm_f32.hip) and the
// last one of a model with its loss (gemm_f32_head.hip).
#ifndef DYNB_GEMM_F32_PRODUCT_H
#define DYNB_GEMM_F32_PRODUCT_H

#include <hip/hip_runtime.h>

#include <type_traits>

#include "dynb_internal.h"
#include "lds_async.h"
#include "softmax_head.h"
#include "tile_map.h"

namespace dynb {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr uint32_t KB = 1024;   // bytes of one copy

// Wait until at most N of this wave's copies (issued last) are pending.
template <int N>
__device__ inline void wait_pending() {
  static_assert(N <= 63, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Wait until every LDS read issued so far has returned: a slot may then be copied into again.  (A copy's
// LDS write is not ordered behind reads in flight, and the compiler waits for these only where their
// values are used.)  The builtin, so that the compiler knows and does not wait for them once more.
__device__ inline void wait_reads() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xc07f);      // lgkmcnt(0), the other counters at their limits
  asm volatile("" ::: "memory");
}

// Forward and input gradient: C[i][j] = sum_k A[i][k] B[j][k], both operands contiguous in k.  A
// block is 32 reduction indices, the whole 128-byte line of each operand row (half a line per block
// fetches every line twice: 19 instead of 11 us at 785 x 301 x 832): two copies of 8 rows per 16 rows.  Granule e
// (16 bytes) of row r sits at slot e ^ (r / 2 % 8), so that matrix instruction e, which reads index
// 4e + kg of 16 rows, finds 64 different banks.
// What bounds it is one wave's chain, whatever the number of tiles: each matrix instruction adds to the last one's
// result, 33 clocks apart.  Scalar instructions, two LDS reads or two copies between two of them are free; one vector
// instruction in between costs 16 clocks, every further one 4 (the result is no longer handed on inside the matrix
// pipe), and more reads or copies cost as much.  So the loop of single tiles has no vector
// instruction at all: the ring is unrolled, its slots are constants in the reads, and the copies' addresses are a
// fixed offset per lane and a scalar base that moves on.  A step of 8 matrix instructions: 548 -> 285 clocks;
// 256 x 512 x 3072 27.4 -> 17 us, 785 x 301 x 832 (where four waves of a compute unit ask for
// more copies than it takes, 23 clocks each) 13.1 -> 8.3.  (The four chains of 2 x 2 tiles have vector
// instructions between them for nothing; there, two steps in a rolled loop.)
// Against 64 x 64 vector-unit tiles: 256 x 512 x 3072 165 us, 785 x 301 x 832 49.
// With HeadArgs (forward, at most 16 columns) the tile's rows of logits go through the softmax and the loss in
// LDS instead of to memory.
template <int MODE, int R, typename Head>
__global__ __launch_bounds__(64) void gemm_f32_kernel(GemmArgs p, Head head) {
  // (40 KB either way: four waves on a compute unit, one per SIMD.  Four blocks of 2 x 2 tiles left room
  // for a fifth wave, and launches of many waves went in uneven rounds: 1024 x 1024 x 4096 134 -> 100
  // us, 2048 x 2048 x 4096 457 -> 354)
  constexpr int NB = R == 1 ? 10 : 5, S = 16 * R;               // S: tile side
  constexpr int G = 2 * R, C = 2 * G;                           // 16-row groups and copies per block
  constexpr uint32_t SLOT = C * KB;
  __shared__ uint4 ring_area[NB * SLOT / 16];
  int ti, tj;
  tile_of_block(blockIdx.x, (p.M + S - 1) / S, (p.N + S - 1) / S, ti, tj);
  const int lane = threadIdx.x, l15 = lane & 15, kg = lane >> 4;
  const int i0 = ti * S, j0 = tj * S;
  const uint32_t lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)&ring_area[0];
  // copy 2g + h: rows 8h .. 8h+7 of group g (g < R: A rows, else B rows); this lane's 16 bytes of
  // the next block, from the tile's first row of the operand (rows past the edge repeat the last one;
  // their products are not stored)
  const char* base[2] = {(const char*)((const float*)p.A + (int64_t)i0 * p.lda),
                         (const char*)((const float*)p.B + (int64_t)j0 * p.ldb)};
  const char* src[C];
  uint32_t off[C];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int g = c >> 1, r = 8 * (c & 1) + (lane >> 3), e = (lane & 7) ^ ((r >> 1) & 7);
    const int i = 16 * g + r, j = 16 * (g - R) + r;
    const int64_t o = g < R ? (i0 + i < p.M ? i : p.M - 1 - i0) * p.lda : (j0 + j < p.N ? j : p.N - 1 - j0) * p.ldb;
    src[c] = base[c / (2 * R)] + (o + 4 * e) * 4;
    off[c] = (uint32_t)(o + 4 * e) * 4;    // (single tiles: fits, see product_side())
  }
  const int blocks = p.K / 32;
  uint32_t ahead = 0;                      // byte offset the next block is copied from; past the end
                                           // the last block is copied again, never used
  auto issue_one = [&](uint32_t slot, int c) {
    if constexpr (R == 1) async_copy_1k_from(base[c / 2], off[c], lds + slot + c * KB);
    else async_copy_1k(src[c] + ahead, lds + slot + c * KB);
  };
  int issued = 0;
  auto advance = [&]() {
    const uint32_t by = ++issued < blocks ? 128 : 0;
    if constexpr (R == 1) { base[0] += by; base[1] += by; }
    else ahead += by;
  };
  uint32_t at[8];                          // this lane's element of granule e of a row group
#pragma unroll
  for (int e = 0; e < 8; ++e) at[e] = (uint32_t)(l15 * 128 + ((e ^ ((l15 >> 1) & 7)) * 16) + 4 * kg);
  float f[2][G][8];                        // [register set][row group][matrix instruction]
  const char* const ring = (const char*)&ring_area[0];
  auto fetch_one = [&](int set, uint32_t slot, int e) {
    const char* const a = ring + (slot + at[e]);
#pragma unroll
    for (int g = 0; g < G; ++g) f[set][g][e] = *(const float*)(a + g * 2048);
  };
  f32x4 acc[R][R];
#pragma unroll
  for (int u = 0; u < R; ++u)
#pragma unroll
    for (int w = 0; w < R; ++w) acc[u][w] = f32x4{0.f, 0.f, 0.f, 0.f};
  constexpr bool HEAD = std::is_same_v<Head, HeadArgs>;
  int label = 0, owned = 1;                // of the row of this lane behind the product: lane / 4
  if constexpr (HEAD) label = head.y[i0 + (lane >> 2) < p.M ? i0 + (lane >> 2) : p.M - 1];
#pragma unroll
  for (int s = 0; s < NB; ++s) {
#pragma unroll
    for (int c = 0; c < C; ++c) issue_one(s * SLOT, c);
    advance();
  }
  if constexpr (HEAD) owned = rows_of_owner(head.segs, i0 + (lane >> 2));
  wait_pending<(NB - 1) * C>();
#pragma unroll
  for (int e = 0; e < 8; ++e) fetch_one(0, 0, e);
  // Step: block c's operands are in registers, or on their way there since the first half of the last
  // step; those of block c + 1 have landed once at most the NB - 2 blocks behind it are pending; block
  // c's slot, whose reads are waited for before this step's own begin, takes block c + NB.
  auto step = [&](int set, uint32_t slot, uint32_t next) {
    wait_pending<(NB - 2) * C>();
#pragma unroll
    for (int e = 0; e < 8; ++e) {
#pragma unroll
      for (int u = 0; u < R; ++u)
#pragma unroll
        for (int w = 0; w < R; ++w)
          acc[u][w] = __builtin_amdgcn_mfma_f32_16x16x4f32(f[set][u][e], f[set][R + w][e], acc[u][w], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (e == 0) wait_reads();
      if (e < 4) {
        fetch_one(set ^ 1, next, 2 * e);
        fetch_one(set ^ 1, next, 2 * e + 1);
      } else if (R > 1 || e < 6) {
        constexpr int PER = R == 1 ? 2 : C / 4;
#pragma unroll
        for (int c = (e - 4) * PER; c < (e - 3) * PER; ++c) issue_one(slot, c);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    advance();
  };
  if constexpr (R == 1) {
    static_assert(NB % 2 == 0, "register sets");
#pragma unroll 1
    for (int c = 0; c < blocks;) {         // (an even number, see launch_gemm_f32())
#pragma unroll
      for (int s = 0; s < NB; s += 2) {
        step(0, s * SLOT, (s + 1) * SLOT);
        step(1, (s + 1) * SLOT, (s + 2) % NB * SLOT);
        c += 2;
        if (c >= blocks) break;
      }
    }
  } else {
    // (two steps unrolled, not the ring: such launches are so short that fetching a long loop body
    // for the first time shows)
    uint32_t slot = 0;
    auto rolled = [&](int set) {
      const uint32_t next = slot + SLOT == NB * SLOT ? 0 : slot + SLOT;
      step(set, slot, next);
      slot = next;
    };
#pragma unroll 1
    for (int c = 0; c < blocks; c += 2) {
      rolled(0);
      rolled(1);
    }
  }
  wait_pending<0>();                       // (no copy may land after the LDS has been given back)

  // accumulator element v of a lane: row 4 * kg + v, column l15
  if constexpr (HEAD) {
    constexpr int PITCH = 20;
    float* const logits = (float*)&ring_area[0];
    wait_reads();                          // (a wave of its own: no barrier)
    const float bias = p.bias ? p.bias[l15 < p.N ? l15 : p.N - 1] : 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float v = acc[0][0][e];
      if (p.bias) v += bias;
      if (p.relu) v = fmaxf(v, 0.f);
      logits[(4 * kg + e) * PITCH + l15] = v;
    }
    __builtin_amdgcn_wave_barrier();
    const int r = lane >> 2, c0 = 4 * (lane & 3);
    const float* const row = logits + r * PITCH;
    const f32x4 z = *(const f32x4*)(row + c0);
    float e[4] = {z[0], z[1], z[2], z[3]};
    const int want = label < 0 ? 0 : label >= p.N ? p.N - 1 : label;   // keeps the read in bounds
    const float loss = softmax_row(4, e, c0, p.N, want, row[want], owned);
    if (i0 + r >= p.M) return;
    float* const dz = (float*)head.dz + (int64_t)(i0 + r) * head.ldd + c0;
    *(f32x4*)dz = f32x4{e[0], e[1], e[2], e[3]};
#pragma unroll
    for (int u = 1; u < 4; ++u) *(f32x4*)(dz + 16 * u) = f32x4{0.f, 0.f, 0.f, 0.f};
    if ((lane & 3) == 0) head.rowloss[i0 + r] = loss;
    return;
  }
#pragma unroll
  for (int w = 0; w < R; ++w) {
    const int j = j0 + 16 * w + l15;
    if (j >= p.N) continue;
    const float bias = MODE == MODE_FWD && p.bias ? p.bias[j] : 0.f;
#pragma unroll
    for (int u = 0; u < R; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = i0 + 16 * u + 4 * kg + e;
        if (i >= p.M) continue;
        float v = acc[u][w][e];
        if (MODE == MODE_FWD) {
          if (p.bias) v += bias;
          if (p.relu) v = fmaxf(v, 0.f);
          if (p.Cf) p.Cf[(int64_t)i * p.ldcf + j] = v;
        } else if (p.mask && !(((const float*)p.mask)[(int64_t)i * p.ldmask + j] > 0.f)) {
          v = 0.f;
        }
        if (p.C) ((float*)p.C)[(int64_t)i * p.ldc + j] = v;
      }
  }
}

}  // namespace
}  // namespace dynb

#endif
