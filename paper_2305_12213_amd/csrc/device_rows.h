// Device helpers for kernels that walk row-major bf16 tensors [rows][ld] with 16-byte
// accesses: a lane takes 8 neighbouring channels of a row, LPR lanes a line of 8 LPR channels (LPR = 8: 128
// bytes; 4: the 64-byte rows of narrow tensors), the 32 LPR threads of a workgroup 32 rows per pass
// (channel granule = tid % LPR, row-lane = tid / LPR).
#ifndef DYNB_DEVICE_ROWS_H
#define DYNB_DEVICE_ROWS_H

#include <hip/hip_runtime.h>

namespace dynb {

typedef __bf16 bf16;

__device__ inline void unpack8(const uint4& q, float (&f)[8]) {
  f[0] = __uint_as_float(q.x << 16); f[1] = __uint_as_float(q.x & 0xffff0000u);
  f[2] = __uint_as_float(q.y << 16); f[3] = __uint_as_float(q.y & 0xffff0000u);
  f[4] = __uint_as_float(q.z << 16); f[5] = __uint_as_float(q.z & 0xffff0000u);
  f[6] = __uint_as_float(q.w << 16); f[7] = __uint_as_float(q.w & 0xffff0000u);
}

__device__ inline uint32_t pack2(float a, float b) {      // round to nearest even, both halves
  const bf16 x = (bf16)a, y = (bf16)b;
  return (uint32_t)__builtin_bit_cast(unsigned short, x) |
         ((uint32_t)__builtin_bit_cast(unsigned short, y) << 16);
}

__device__ inline uint4 pack8(const float (&f)[8]) {
  return make_uint4(pack2(f[0], f[1]), pack2(f[2], f[3]), pack2(f[4], f[5]), pack2(f[6], f[7]));
}

// Mask of 8 neighbouring channels of which the first `live` exist (any value): padding channels are
// stored as zeros whatever the data -- a product with zero weights is no zero next to an infinity.
__device__ inline uint4 keep8(int live) {
  auto word = [&](int d) { return live > 2 * d + 1 ? 0xffffffffu : live > 2 * d ? 0x0000ffffu : 0u; };
  return make_uint4(word(0), word(1), word(2), word(3));
}
// Mask of those of 8 values that are > 0 (a ReLU's gradient passes where its output is).
__device__ inline uint4 positive8(const uint4& q) {
  float k[8];
  unpack8(q, k);
  auto word = [&](int d) { return (k[2 * d] > 0.f ? 0x0000ffffu : 0u) | (k[2 * d + 1] > 0.f ? 0xffff0000u : 0u); };
  return make_uint4(word(0), word(1), word(2), word(3));
}
__device__ inline uint4 operator&(const uint4& a, const uint4& b) {
  return make_uint4(a.x & b.x, a.y & b.y, a.z & b.z, a.w & b.w);
}

__device__ inline uint4 load8(const bf16* p) { return *reinterpret_cast<const uint4*>(p); }
__device__ inline void store8(bf16* p, const uint4& q) { *reinterpret_cast<uint4*>(p) = q; }

// Granule (16 bytes) g of a 128-byte row r in LDS sits at slot g ^ swizzle128(r): 16 neighbouring rows, read at
// one granule, then fall into 64 different banks (two rows per pass over the banks; rows r and r + 8
// differ in the lowest bit, which also keeps lanes l and l + 32 apart).
__device__ inline int swizzle128(int r) { return (((r >> 1) & 3) << 1) | ((r >> 3) & 1); }

// This lane's granules of the first n >= 1 of 32 F rows: rows row-lane + 32 i.  Rows past the last repeat it,
// so that no branch stands between the loads and all are in flight together; the address is one uniform
// base and a 32-bit offset (256 rows of a tensor below 2 GiB).
constexpr int ROWS_IN_FLIGHT = 8;          // per lane, at most
template <int LPR, int F>
__device__ inline void load_rows(const bf16* base, int64_t ld, int n, uint4 (&q)[F]) {
  static_assert(F <= ROWS_IN_FLIGHT, "32-bit offsets");
  const uint32_t pitch = (uint32_t)ld * 2, g = (threadIdx.x % LPR) * 16;
  const int rl = threadIdx.x / LPR;
#pragma unroll
  for (int i = 0; i < F; ++i)
    q[i] = *(const uint4*)((const char*)base + ((uint32_t)min(rl + 32 * i, n - 1) * pitch + g));
}

// Sums a[0..7] (this lane's 8 channels) over the 32 row-lanes of the workgroup, in a fixed order (the same for
// every LPR): eight neighbouring row-lanes as a tree, then the four groups of eight in turn; `red` is
// workgroup-shared.  Each exchange between lanes halves the channels that a lane still carries (7 exchanges
// instead of the 24 of whole vectors), so that a lane ends with one channel of its group.
template <int LPR>
__device__ inline void sum_over_row_group(const float (&a)[8], float (*red)[8 * LPR]) {
  const int t = threadIdx.x;
  const bool u = t & LPR, v = t & (2 * LPR), w = t & (4 * LPR);
  float b[4], c[2];
#pragma unroll
  for (int j = 0; j < 4; ++j) b[j] = (u ? a[j + 4] : a[j]) + __shfl_xor(u ? a[j] : a[j + 4], LPR);
#pragma unroll
  for (int j = 0; j < 2; ++j) c[j] = (v ? b[j + 2] : b[j]) + __shfl_xor(v ? b[j] : b[j + 2], 2 * LPR);
  red[t / (8 * LPR)][(t % LPR) * 8 + (u ? 4 : 0) + (v ? 2 : 0) + (w ? 1 : 0)] =
      (w ? c[1] : c[0]) + __shfl_xor(w ? c[0] : c[1], 4 * LPR);
}

// ... every thread ends with the totals of its channels
template <int LPR>
__device__ inline void sum_over_rows(float (&a)[8], float (*red)[8 * LPR]) {
  const int cg = threadIdx.x % LPR;
  __syncthreads();
  sum_over_row_group<LPR>(a, red);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 8; ++j)
    a[j] = ((red[0][cg * 8 + j] + red[1][cg * 8 + j]) + red[2][cg * 8 + j]) + red[3][cg * 8 + j];
}

// ... the total of channel threadIdx.x, for the first 8 LPR threads
template <int LPR>
__device__ inline float channel_sum(const float (&a)[8], float (*red)[8 * LPR]) {
  const int c = threadIdx.x % (8 * LPR);
  __syncthreads();
  sum_over_row_group<LPR>(a, red);
  __syncthreads();
  return ((red[0][c] + red[1][c]) + red[2][c]) + red[3][c];
}

}  // namespace dynb

#endif
