// kt_skinny.h -- Y = X R for a handful of tokens (a decode step): bf16 X, at most 64 rows.
//
// With so few tokens the call is the read of R: the general path transposes and rounds all of R (one read, one
// write), reads that copy again and has d / 256 output tiles, i.e. at d = 4096 sixteen workgroups walking K alone.
// Here R is read once, as it is: a workgroup takes 64 of its columns and a range of its rows, each wave 64 rows at
// a time (256-byte row pieces, 16 KiB in flight per wave and the next 16 KiB behind them), rounds them to bf16
// into its own 8 KiB of LDS and multiplies from there, K as the row index of the LDS tile (transposing reads).
// The four waves add up in LDS, the row ranges (grid.y) in splitk_reduce_kernel, both in fixed order.
// Bound: HBM, 4 d^2 bytes of an fp32 R.
#pragma once
#include "kt_aux.h"

namespace kt {

constexpr int kSkinnyMaxTokens = 64;

// TB: blocks of 16 tokens.  grid = (d / 64, row ranges of k_per_wg, problems).  Rows of R 16-byte aligned.
// part[range * split_stride + (problem * n + token) * d + column]
template <typename TR, int TB>
__global__ __launch_bounds__(256) void skinny_rotate_kernel(const __bf16* __restrict__ X, int64_t ldx,
                                                            int64_t x_batch_stride, const TR* __restrict__ R,
                                                            int64_t ldr, int n, int d, int k_per_wg,
                                                            float* __restrict__ part, int64_t split_stride) {
  constexpr int ROWS = 64;                                  // rows of R per wave and round
  constexpr int VEC = 16 / (int)sizeof(TR);                 // columns per 16-byte load
  constexpr int LPR = 64 / VEC;                             // lanes per row of 64 columns
  constexpr int NLD = ROWS * LPR / 64;
  __shared__ __align__(16) char lds_all[4 * ROWS * 128];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, q = lane >> 4;
  char* lds = lds_all + wave * (ROWS * 128);
  X += (int64_t)blockIdx.z * x_batch_stride;
  R += (int64_t)blockIdx.z * d * ldr + blockIdx.x * 64;
  const int k_begin = blockIdx.y * k_per_wg;
  const int k_end = k_begin + k_per_wg < d ? k_begin + k_per_wg : d;  // multiples of 64

  // 32-byte pieces of a tile row (128 bytes) are XOR-swizzled so that the rows two lane quarters read together
  // (k .. k+3 and k+8 .. k+11, one piece) hit different banks
  auto piece_key = [](int row) __attribute__((always_inline)) { return ((row >> 1) & 1) | (((row >> 3) & 1) << 1); };
  const int lrow = lane / LPR, lcol = (lane % LPR) * VEC;   // row and first column of load 0; load i: + i (64 / LPR) rows
  intx4 cur[NLD], nxt[NLD];
  auto request = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NLD; ++i)
      if (k0 < k_end) nxt[i] = *reinterpret_cast<const intx4*>(R + (int64_t)(k0 + lrow + i * (64 / LPR)) * ldr + lcol);
  };
  floatx4 acc[TB][4];
#pragma unroll
  for (int t = 0; t < TB; ++t)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[t][c] = floatx4{0.f, 0.f, 0.f, 0.f};

  request(k_begin + wave * ROWS);
#pragma unroll 1
  for (int k0 = k_begin + wave * ROWS; k0 < k_end; k0 += 4 * ROWS) {
    intx4 xa[2][TB];  // X fragments: token l16 of the block, 8 values of K of quarter q
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int t = 0; t < TB; ++t) {
        const int token = 16 * t + l16 < n ? 16 * t + l16 : n - 1;
        xa[h][t] = *reinterpret_cast<const intx4*>(X + (int64_t)token * ldx + k0 + 32 * h + 8 * q);
      }
#pragma unroll
    for (int i = 0; i < NLD; ++i) cur[i] = nxt[i];
    request(k0 + 4 * ROWS);
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int row = lrow + i * (64 / LPR);
      char* dst = lds + row * 128 + (((lcol >> 4) ^ piece_key(row)) << 5) + 2 * (lcol & 15);
      if constexpr (sizeof(TR) == 4) {
        typedef __bf16 bf16x4v __attribute__((ext_vector_type(4)));
        const floatx4 v = __builtin_bit_cast(floatx4, cur[i]);
        const bf16x4v h = {(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
        *reinterpret_cast<bf16x4v*>(dst) = h;
      } else {
        *reinterpret_cast<intx4*>(dst) = cur[i];
      }
    }
    // the tile is the wave's own and LDS operations of one wave complete in order; keep the compiler in order too
    asm volatile("" ::: "memory");
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int row = 32 * h + 8 * q + (l16 >> 2);
        const int addr = row * 128 + ((c ^ piece_key(row)) << 5) + 8 * (l16 & 3);
        const intx4 rb = read_tr_operand(lds, addr, addr + 4 * 128);
#pragma unroll
        for (int t = 0; t < TB; ++t)
          acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, xa[h][t]),
                                                              __builtin_bit_cast(bf16x8, rb), acc[t][c], 0, 0, 0);
      }
    asm volatile("" ::: "memory");
  }

  // the four waves' sums, 16 tokens at a time: red[wave][token][column]
  float* red = reinterpret_cast<float*>(lds_all);
  const int tok = threadIdx.x >> 4, col = (threadIdx.x & 15) * 4;
#pragma unroll
  for (int t = 0; t < TB; ++t) {
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave * 1024 + (4 * q + r) * 64 + 16 * c + l16] = acc[t][c][r];
    __syncthreads();
    const int token = 16 * t + tok;
    if (token < n) {
      floatx4 v = *reinterpret_cast<const floatx4*>(red + tok * 64 + col);
#pragma unroll
      for (int w = 1; w < 4; ++w) v += *reinterpret_cast<const floatx4*>(red + w * 1024 + tok * 64 + col);
      *reinterpret_cast<floatx4*>(part + blockIdx.y * split_stride + ((int64_t)blockIdx.z * n + token) * d + blockIdx.x * 64 + col) = v;
    }
  }
}

}  // namespace kt
