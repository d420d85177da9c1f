// Epilogue of the bf16 forward and input-gradient products on 32 x 32 matrix-instruction tiles.
#ifndef DYNB_GEMM_EPILOGUE_H
#define DYNB_GEMM_EPILOGUE_H

#include <hip/hip_runtime.h>

#include "dynb_internal.h"

namespace dynb {
namespace {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// A wave's results: TM x TN tiles from row i_first and column j_first on; element v of lane l of a tile is
// (row l % 32, column 8 (v / 4) + 4 (l / 32) + v % 4).  Row i of the product is row row_of(i) of the output.
// The strip passes, 32 rows at a time, through a
// private fp32 patch of 32 x (32 TN + 4) floats in LDS: the accumulator layout (4 consecutive columns per lane, 32
// rows per instruction) becomes 8 consecutive columns per lane, 4 to 16 rows per instruction,
// and bias/ReLU/mask, the bf16 conversion and the global accesses run on whole 128-byte
// lines.
template <int MODE, int TM, int TN, typename RowOf>
__device__ __forceinline__ void store_product(const GemmArgs& p, int M, const f32x16 (&acc)[TM][TN], float* patch,
                                              int i_first, int j_first, RowOf row_of) {
  const int lane = threadIdx.x & 63, hi4 = 4 * (lane >> 5), l31 = lane & 31;
  constexpr int CW = 32 * TN;              // columns of the strip
  constexpr int EP = CW + 4;               // patch row pitch in floats
  static_assert(CW == 128 || CW == 64 || CW == 32, "strip width");
  constexpr int LPR = CW / 8;              // lanes per row in the read-back phase
  constexpr int RPI = 64 / LPR;            // rows per read-back instruction
  const int rrow = lane / LPR, rcol = (lane % LPR) * 8;
  const int jcol = j_first + rcol;         // first of the lane's 8 columns
  const bool col_ok = jcol + 7 < p.N;
  const bool bias_vec = (((uintptr_t)p.bias) & 15) == 0;   // a layer's bias may start anywhere
  float bv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (MODE == MODE_FWD && p.bias) {
    if (col_ok && bias_vec) {
      const float4 t0 = *(const float4*)&p.bias[jcol], t1 = *(const float4*)&p.bias[jcol + 4];
      bv[0] = t0.x; bv[1] = t0.y; bv[2] = t0.z; bv[3] = t0.w;
      bv[4] = t1.x; bv[5] = t1.y; bv[6] = t1.z; bv[7] = t1.w;
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (jcol + e < p.N) bv[e] = p.bias[jcol + e];
    }
  }
  // input gradient: the mask and addend rows of a 32-row block are asked for one block ahead, all of
  // them at once (rows past the matrix clamped), and travel while the accumulators pass
  // through the patch -- fetched row by row where they are used, every row costs a trip to
  // memory of its own, and block by block every block one
  bf16x8 mkv[2][32 / RPI], adv[2][32 / RPI];
  auto ask = [&](int a) {
    if (MODE != MODE_DGRAD || !col_ok) return;
#pragma unroll
    for (int t = 0; t < 32 / RPI; ++t) {
      int i = i_first + a * 32 + rrow + RPI * t;
      i = row_of(i < M ? i : M - 1);
      if (p.mask) mkv[a & 1][t] = *(const bf16x8*)((const bf16*)p.mask + (int64_t)i * p.ldmask + jcol);
      if (p.addend) adv[a & 1][t] = *(const bf16x8*)((const bf16*)p.addend + (int64_t)i * p.ldadd + jcol);
    }
  };
  ask(0);
#pragma unroll
  for (int a = 0; a < TM; ++a) {
    if (a + 1 < TM) ask(a + 1);
#pragma unroll
    for (int b = 0; b < TN; ++b)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 o = {acc[a][b][4 * q], acc[a][b][4 * q + 1], acc[a][b][4 * q + 2],
                         acc[a][b][4 * q + 3]};
        *(f32x4*)&patch[l31 * EP + b * 32 + 8 * q + hi4] = o;
      }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int t = 0; t < 32 / RPI; ++t) {
      const int r = rrow + RPI * t;
      int i = i_first + a * 32 + r;
      const f32x4 lo = *(const f32x4*)&patch[r * EP + rcol];
      const f32x4 hi = *(const f32x4*)&patch[r * EP + rcol + 4];
      if (i >= M || jcol >= p.N) continue;
      i = row_of(i);
      float v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      if (MODE == MODE_FWD) {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += bv[e];
        if (p.relu) {
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = fmaxf(v[e], 0.f);
        }
      }
      if (col_ok) {
        if (MODE == MODE_DGRAD && p.addend) {
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = (float)(bf16)v[e] + (float)adv[a & 1][t][e];
        }
        if (MODE == MODE_DGRAD && p.mask) {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (!((float)mkv[a & 1][t][e] > 0.f)) v[e] = 0.f;
        }
        if (MODE == MODE_FWD && p.Cf) {
          float* dst = p.Cf + (int64_t)i * p.ldcf + jcol;
          *(float4*)dst = make_float4(v[0], v[1], v[2], v[3]);
          *(float4*)(dst + 4) = make_float4(v[4], v[5], v[6], v[7]);
        }
        if (p.C) {
          const bf16x8 o = {(bf16)v[0], (bf16)v[1], (bf16)v[2], (bf16)v[3],
                            (bf16)v[4], (bf16)v[5], (bf16)v[6], (bf16)v[7]};
          *(bf16x8*)((bf16*)p.C + (int64_t)i * p.ldc + jcol) = o;
        }
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int j = jcol + e;
          if (j >= p.N) continue;
          float w = v[e];
          if (MODE == MODE_DGRAD && p.addend)
            w = (float)(bf16)w + (float)((const bf16*)p.addend)[(int64_t)i * p.ldadd + j];
          if (MODE == MODE_DGRAD && p.mask &&
              !((float)((const bf16*)p.mask)[(int64_t)i * p.ldmask + j] > 0.f))
            w = 0.f;
          if (MODE == MODE_FWD && p.Cf) p.Cf[(int64_t)i * p.ldcf + j] = w;
          if (p.C) ((bf16*)p.C)[(int64_t)i * p.ldc + j] = (bf16)w;
        }
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
}

}  // namespace
}  // namespace dynb

#endif
