// kt_gemm32.h -- fp32 products of few tiles: 32 x 32 per workgroup, operands straight from memory into registers.
//
// The fp32 matrix pipe of a CU does 256 flop per cycle, so a 64 x 64 tile of the LDS loop takes 1024 cycles per 32 of K: 64
// tiles, a 512 x 512 product, keep 64 of 256 CUs busy for K / 32 x 0.45 us.  Here a tile is a quarter of that and its four
// waves share K (chunks of 32 in turn), so that the same product is 256 workgroups of K / 128 steps.
// A step (32 of K) is 32 matrix instructions on 8 KiB of operands, which come through the caches directly in the form the
// instruction takes them: no LDS round trip, no barrier, three steps in flight.  The four sums meet in LDS in fixed order.
//
// Bound: the L2, 32 bytes a cycle and CU (8 KiB in 256 matrix cycles), twice what the 64 x 64 tiles read; those win where they fill the chip.
#pragma once
#include "kt_gemm.h"

namespace kt {

using TF_32 = Tile<float, 32, 32, 2, 2>;
constexpr int k32Pitch = 36;  // floats per row of a wave's sums in LDS
static_assert(4 * 32 * k32Pitch * 4 <= TF_32::LDS_BYTES, "the four sums fit the LDS the tile type reserves");

// acc = this wave's 16 x 16 block (Frag<TF_32>) of A B^T over K = [k0, k1), a multiple of 128.  AT / BT: the operand has K as its
// row index; M (N) is then a multiple of 4, and rows of A beyond k_valid are read from the last valid one.
template <bool AT, bool BT, bool SWAP>
__device__ __forceinline__ void gemm32_mainloop(const float* A, int64_t lda, int M, int m0, const float* B, int64_t ldb, int N, int n0,
                                                int k0, int k1, floatx4 (&acc)[1][1], char* lds, int k_valid) {
  const Frag<TF_32> f;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  struct Step { floatx4 a[2][2], b[2][2]; };  // [block of 16][16 of K], four values of K of this lane's row

  // K along the rows: lane (l16, q) takes 16 bytes at K = 4 q of rows l16 and l16 + 16 of the tile.  K as the row index: 8 bytes
  // at columns 2 l16, 2 l16 + 1 of rows 4 q .. 4 q + 3; block i of the tile is then the columns 2 l16 + i.
  uint32_t oa[AT ? 1 : 2], ob[BT ? 1 : 2];
  auto offsets = [&](auto t_c, uint32_t* o, int64_t ld, int size, int first) __attribute__((always_inline)) {
    if constexpr (decltype(t_c)::value) {
      const int c = 2 * f.l16 < size - first ? 2 * f.l16 : size - first - 2;
      o[0] = (uint32_t)((4 * f.q * ld + c) * 4);
    } else {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        int row = 16 * i + f.l16;
        row = first + row < size ? row : size - 1 - first;
        o[i] = (uint32_t)((row * ld + 4 * f.q) * 4);
      }
    }
  };
  offsets(std::integral_constant<bool, AT>{}, oa, lda, M, m0);
  offsets(std::integral_constant<bool, BT>{}, ob, ldb, N, n0);
  const char* Ab = reinterpret_cast<const char*>(AT ? A + m0 : A + (int64_t)m0 * lda);
  const char* Bb = reinterpret_cast<const char*>(BT ? B + n0 : B + (int64_t)n0 * ldb);

  auto load_operand = [&](auto t_c, floatx4 (&v)[2][2], const char* base, const uint32_t* o, int64_t ld, int k, int rows) __attribute__((always_inline)) {
    if constexpr (decltype(t_c)::value) {
      const char* p = base + (int64_t)k * ld * 4;
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          uint32_t at = o[0] + (uint32_t)((16 * h + e) * ld * 4);
          if (k + 32 > rows) {  // (uniform) the last rows: none beyond `rows`, which may lie before k
            const int row = k + 16 * h + 4 * f.q + e < rows ? 16 * h + e : rows - 1 - k - 4 * f.q;
            const float2 w = *reinterpret_cast<const float2*>(p + (int64_t)o[0] + (int64_t)row * ld * 4);
            v[0][h][e] = w.x; v[1][h][e] = w.y;
          } else {
            const float2 w = *reinterpret_cast<const float2*>(p + at);
            v[0][h][e] = w.x; v[1][h][e] = w.y;
          }
        }
    } else {
      const char* p = base + (int64_t)k * 4;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) v[i][h] = *reinterpret_cast<const floatx4*>(p + o[i] + 64 * h);
    }
  };
  const int steps = (k1 - k0) >> 7;  // of this wave
  auto load = [&](Step& s, int n) __attribute__((always_inline)) {
    const int k = k0 + 128 * n + 32 * wave;
    load_operand(std::integral_constant<bool, AT>{}, s.a, Ab, oa, lda, k, AT ? k_valid : 0x7fffffff);
    load_operand(std::integral_constant<bool, BT>{}, s.b, Bb, ob, ldb, k, 0x7fffffff);
  };
  floatx4 c[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) c[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  int n = 0;
  auto step = [&](Step& s) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) c[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(s.a[i][h][e], s.b[j][h][e], c[i][j], 0, 0, 0);
    if (n + 3 < steps) load(s, n + 3);
    return ++n < steps;
  };
  Step s0, s1, s2;
  load(s0, 0);
  if (steps > 1) load(s1, 1);
  if (steps > 2) load(s2, 2);
  while (step(s0) && step(s1) && step(s2)) {}

  float* red = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = AT ? 2 * (4 * f.q + r) + i : 16 * i + 4 * f.q + r, nn = BT ? 2 * f.l16 + j : 16 * j + f.l16;
        red[(32 * wave + m) * k32Pitch + nn] = c[i][j][r];
      }
  __syncthreads();
  auto sum = [&](auto at) __attribute__((always_inline)) { return ((at(0) + at(1)) + at(2)) + at(3); };
  if constexpr (SWAP) {
    const float* p = red + f.m_row(0) * k32Pitch + f.n_quad(0);
    acc[0][0] = sum([&](int w) __attribute__((always_inline)) { return *reinterpret_cast<const floatx4*>(p + w * 32 * k32Pitch); });
  } else {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float* p = red + f.m_of(0, r) * k32Pitch + f.n_of(0);
      acc[0][0][r] = sum([&](int w) __attribute__((always_inline)) { return p[w * 32 * k32Pitch]; });
    }
  }
}

template <class Epi, bool AT, bool BT>
__global__ __launch_bounds__(256) void gemm32_kernel(GemmShape g, Epi epi) {
  extern __shared__ __align__(16) char lds[];
  const int batch = blockIdx.y;
  int tm, tn, ks;
  if (!tile_of_block(g, tm, tn, ks)) return;
  if (epi.skip(batch)) return;
  const int slab0 = ks * g.slabs_per_split;
  const int slab1 = slab0 + g.slabs_per_split < g.slabs_total ? slab0 + g.slabs_per_split : g.slabs_total;
  floatx4 acc[1][1];
  gemm32_mainloop<AT, BT, Epi::kSwap>(static_cast<const float*>(g.A) + (int64_t)batch * g.batch_stride_a, g.lda, g.M, tm * 32,
                                      static_cast<const float*>(g.B) + (int64_t)batch * g.batch_stride_b, g.ldb, g.N, tn * 32, 32 * slab0,
                                      32 * slab1, acc, lds, g.k_valid);
  epi(acc, batch, tm, tn, ks, tm * 32, tn * 32);
}

}  // namespace kt
