// kt_fused_d128.h -- the whole loss + gradient pass for head-dimension rotations
// (d = 128, bf16) in ONE kernel that reads X exactly once.
//
// For many small independent problems (one 128 x 128 rotation per KV head and layer, the
// R2 learner of "Learning the Rotations") the path of one product after the other is
// bandwidth-bound: it reads X twice and writes and re-reads Y and dL/dY.  Here a workgroup
// walks token tiles of 128 rows of one problem and, per tile,
//   B. Y = X_tile R            (MFMA; token on the lane, all 128 features of a token in the
//                               registers of four lanes)
//   C. per-token mean, centred moments (two-pass, fp32), kurtosis, loss term,
//      coefficients           (Eq. 3 and its chain rule; Y is still in registers: no recompute)
//   D. G = dL/dY -> bf16 -> LDS, token-major like the X tile
//   E. dR += X_tile^T G_tile   (MFMA; both operands are read token-minor straight out of the
//                               token-major LDS tiles with ds_read_b64_tr_b16, the gfx950
//                               transposing LDS read)
// and keeps its 128 x 128 share of dR in registers until its last tile.
// Partial dR and loss sums of the workgroups of a problem are added by fixed-order
// reduction kernels afterwards.
//
// LDS (160 KiB): three X tiles and two G tiles of 32 KiB, rows of 256 bytes; R^T lives in registers.
//  X: 16-byte chunks XOR-swizzled with xkey(row) = 4*(row%4) + (row/4)%4: distinct over 16 consecutive rows (conflict-free
//  16-byte fragment reads of 16 rows at one column), and the rows k..k+3, k+8..k+11 that two lane quarters read transposed,
//  32 bytes each, fall into eight different 32-byte bank groups.
//  G: 8-byte units XOR-swizzled with gkey(t) = 2*p(t), p a permutation of 0..15: two neighbouring units of 16 tokens are
//  distinct (conflict-free 8-byte stores of two lane quarters), and p/2 is distinct over the eight rows of a transposed read.
#pragma once
#include "kt_aux.h"
#include "kt_gemm.h"

namespace kt {

constexpr int kF128Tile = 128;                  // tokens per tile
constexpr int kF128BufBytes = kF128Tile * 256;  // one X or G tile: 128 rows of 256 bytes
constexpr int kF128GOff = 3 * kF128BufBytes;     // LDS: X[3] | G[2]
constexpr int kF128LdsBytes = 5 * kF128BufBytes;  // 160 KiB

__device__ __forceinline__ int f128_xkey(int row) { return ((row & 3) << 2) | ((row >> 2) & 3); }
__device__ __forceinline__ int f128_gkey(int t) { return ((t & 3) << 3) | ((t & 8) >> 1) | ((t & 4) >> 1); }

// The matrix-core instructions of this kernel are written as inline assembly so that the
// register file of every operand is fixed: R^T fragments live in accumulation registers (only
// the matrix core touches them), everything else in vector registers.  Left to the register
// allocator the registers of R^T get shuffled between the two files every tile.
// The compiler does not know these are matrix instructions: results are read by other
// instruction types only behind mfma16_result_fence().
__device__ __forceinline__ void mfma16_y_first(floatx4& y, const intx4& rt, const intx4& x) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(y) : "a"(rt), "v"(x));
}
__device__ __forceinline__ void mfma16_y(floatx4& y, const intx4& rt, const intx4& x) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(y) : "a"(rt), "v"(x));
}
__device__ __forceinline__ void mfma16_result_fence(floatx4 (&y)[8]) {
  asm volatile("s_nop 15" : "+v"(y[0]), "+v"(y[1]), "+v"(y[2]), "+v"(y[3]), "+v"(y[4]), "+v"(y[5]), "+v"(y[6]), "+v"(y[7]));
}
__device__ __forceinline__ void mfma16_dr(floatx4& acc, const intx4& xt, const intx4& gt) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(xt), "v"(gt));
}
__device__ __forceinline__ void mfma16_result_fence(floatx4 (&a)[2][4]) {
  asm volatile("s_nop 15" : "+v"(a[0][0]), "+v"(a[0][1]), "+v"(a[0][2]), "+v"(a[0][3]), "+v"(a[1][0]), "+v"(a[1][1]), "+v"(a[1][2]), "+v"(a[1][3]));
}

// 16 bytes per lane from global memory straight into LDS: lane l lands at lds_addr + 16 l
// (lds_addr is wave-uniform).  Written as assembly so that the compiler does not tie later LDS
// reads to these loads with a full wait; the waits are placed by hand (vmcnt).
// Source: a wave-uniform base (from scalar instructions) and 32 bits of byte offset per lane.
__device__ __forceinline__ void load_to_lds_16(uint32_t voffset, const char* base, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voffset), "s"(base), "s"(lds_addr)
               : "memory", "m0");
}

// One problem's R (row-major, fp32 or bf16, any alignment) rounded to bf16 into a swizzled 128 x 256-byte LDS tile, K as the
// row: what fragments of R^T are read from (transposing reads), so that no launch has to write R^T first.  8 bytes a step.
template <int NT>
__device__ __forceinline__ void stage_rotation(const void* __restrict__ R, int64_t ldr, int r_bf16, char* tile) {
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  const bool vec = ((reinterpret_cast<uintptr_t>(R) | (uintptr_t)(ldr * (r_bf16 ? 2 : 4))) & (r_bf16 ? 7 : 15)) == 0;  // uniform
  auto place = [&](int u, bf16x4 v) __attribute__((always_inline)) {
    const int row = u >> 5, c = u & 31;
    *reinterpret_cast<bf16x4*>(tile + row * 256 + (((c >> 1) ^ f128_xkey(row)) << 4) + ((c & 1) << 3)) = v;
  };
  constexpr int N = 128 * 32 / NT;
  if (r_bf16) {
    const __bf16* src = static_cast<const __bf16*>(R);
    bf16x4 v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int u = (int)threadIdx.x + NT * i;
      const __bf16* p = src + (int64_t)(u >> 5) * ldr + 4 * (u & 31);
      if (vec) {
        v[i] = *reinterpret_cast<const bf16x4*>(p);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[i][e] = p[e];
      }
    }
#pragma unroll
    for (int i = 0; i < N; ++i) place((int)threadIdx.x + NT * i, v[i]);
  } else {
    const float* src = static_cast<const float*>(R);
    floatx4 v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int u = (int)threadIdx.x + NT * i;
      const float* p = src + (int64_t)(u >> 5) * ldr + 4 * (u & 31);
      if (vec) {
        v[i] = *reinterpret_cast<const floatx4*>(p);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[i][e] = p[e];
      }
    }
#pragma unroll
    for (int i = 0; i < N; ++i) place((int)threadIdx.x + NT * i, bf16x4{(__bf16)v[i][0], (__bf16)v[i][1], (__bf16)v[i][2], (__bf16)v[i][3]});
  }
}

// grid = (S, batch): S workgroups share the token tiles of one problem.
// dR_part[(wg * batch + b) * 128*128 + k*128 + j], loss_part[b * S + wg].
//
// Eight waves, two per SIMD, 16 tokens of the tile each (16 x 16 matrix blocks: R^T 128 registers, Y 32, a 32 x 64 share of
// dR 32).  Phase i of a workgroup (one barrier each): B - D of its tile i, E of its tile i - 1, the loads of tile i + 1.
// X(i) lives in X buffer i % 3, G(i) in G buffer i & 1.  Waves 0 - 3 run E behind D, waves 4 - 7 ahead of B: of the two waves of a
// SIMD one is at its matrix instructions while the other is at its vector instructions.
//
// What bounds it: the board's power limit (1.4 kW, 1.8 - 1.9 GHz of 2.4; with X out of the caches instead of HBM the same cycles
// run at 2.2 GHz).  256 problems x 131072 tokens (8 GiB, 2.2e12 flop), launches in a row, ms: four waves of 32 tokens with E
// dealt between the vector instructions of C and D 2.95 (5950 cycles a tile, one wave's issue), eight waves in two roles (B -
// D; E and loads) 2.87 (5280), this form 2.73 (4950; 2.83 with E behind D in every wave).  Fewer cycles did not help further:
// E in 32 x 32 blocks, the loads dealt between matrix instructions and independent vector instructions side by side 2.8 - 2.95.
__global__ __launch_bounds__(512) void fused_d128_kernel(const __bf16* __restrict__ X, int64_t ldx,
                                                         int64_t x_batch_stride,
                                                         const void* __restrict__ R, int64_t ldr, int r_bf16, int n,
                                                         float kappa_target,
                                                         float* __restrict__ row_kurt,
                                                         double* __restrict__ loss_part,
                                                         float* __restrict__ dR_part, int want_grad) {
  extern __shared__ __align__(16) char lds[];
  constexpr int D = 128, T = kF128Tile, BUF = kF128BufBytes;
  using std::integral_constant;
  const int b = blockIdx.y, S = gridDim.x, wg = blockIdx.x, batch = gridDim.y;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane >> 4, l16 = lane & 15;
  X += (int64_t)b * x_batch_stride;
  R = static_cast<const char*>(R) + (int64_t)b * D * ldr * (r_bf16 ? 2 : 4);
  const int tiles = (n + T - 1) / T;
  const int my_tiles = wg < tiles ? (tiles - wg + S - 1) / S : 0;  // tiles wg, wg+S, ...

  // X tile movement: a wave owns rows 16 wave .. + 15 of the tile and moves them with 4 instructions of 4 rows (1 KiB)
  // each.  The 16-byte swizzle is applied on the source side: LDS chunk position l16 of row r receives global chunk
  // l16 ^ xkey(r).
  const unsigned lds_wave = (unsigned)(size_t)(__attribute__((address_space(3))) char*)lds + wave * (16 * 256);
  const uint32_t xrow_off = (uint32_t)((wave * 16 + q) * ldx * 2);  // bytes from the tile's first row (ldx <= 2^22)
  auto load_tile = [&](int tile, int buf) __attribute__((always_inline)) {
    const char* src = reinterpret_cast<const char*>(X) + (int64_t)tile * T * ldx * 2;
    auto one = [&](int i) __attribute__((always_inline)) {
      load_to_lds_16(xrow_off + ((l16 ^ f128_xkey(4 * i + q)) << 4), src + (int64_t)(4 * i) * ldx * 2, lds_wave + buf * BUF + i * 1024);
    };
    if (tile * T + T <= n) {
#pragma unroll
      for (int i = 0; i < 4; ++i) one(i);
    } else {  // last, partial tile: rows past the end are zero-filled
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (tile * T + wave * 16 + 4 * i + q < n)
          one(i);
        else
          *reinterpret_cast<intx4*>(lds + buf * BUF + wave * (16 * 256) + i * 1024 + lane * 16) = intx4{0, 0, 0, 0};
      }
    }
  };
  if (my_tiles > 0) load_tile(wg, 0);

  // dR: 32 features of X (rows) x 64 of G (columns) per wave
  const int wm4 = wave >> 1, wn2 = wave & 1;
  floatx4 acc2[2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      acc2[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
  double loss_acc = 0.0;
  const float inv_d = 1.0f / (float)D;
  const float grad_scale = 4.0f / ((float)n * (float)D);

  // lane constants of the transposing reads (stage E): token row 32 s + 8 q + l16 / 4 (+4), 4 features 4 (l16 % 4) of a block of 16
  // (row + 4 and the next block of 16 features: other bits of the address)
  const int tr_row = 8 * q + (l16 >> 2), ux = wm4 * 8 + (l16 & 3), ug = wn2 * 16 + (l16 & 3);  // 8-byte unit of block 0
  int xa = tr_row * 256 + (((ux >> 1) ^ f128_xkey(tr_row)) << 4) + ((ux & 1) << 3);
  int ga = kF128GOff + tr_row * 256 + ((ug ^ f128_gkey(tr_row)) << 3);
  constexpr int kRow4 = 4 * 256 + 16, kBlock = 32;

  // R^T fragments for all 4 K steps and 8 feature blocks: 128 registers, read once from G buffer 1 (first written in
  // phase 1).  From global memory every wave would take 32 KiB through the L1: 2 us of a call of few tiles.
  stage_rotation<512>(R, ldr, r_bf16, lds + kF128GOff + BUF);
  lds_barrier();
  intx4 rtf[4][8];
  const int ra = kF128GOff + BUF + tr_row * 256 + ((((l16 & 3) >> 1) ^ f128_xkey(tr_row)) << 4) + ((l16 & 1) << 3);
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int mb = 0; mb < 8; ++mb) {
      const int at = ra ^ (mb * kBlock);
      rtf[s][mb] = read_tr_operand(lds, at + s * 32 * 256, (at ^ kRow4) + s * 32 * 256);
    }
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int mb = 0; mb < 8; ++mb) asm volatile("" : "+a"(rtf[s][mb]));

  // B, C, D of tile `tile` (X buffer xbuf, G buffer gbuf)
  auto stage_bcd = [&](int tile, int xbuf, int gbuf) __attribute__((always_inline)) {
    floatx4 acc[8];  // Y of token 16 wave + l16 of the tile: features 16 mb + 4 q + r
    {
      const char* xrow = lds + xbuf * BUF + (wave * 16 + l16) * 256;
      intx4 xb[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) xb[s] = *reinterpret_cast<const intx4*>(xrow + (((4 * s + q) ^ f128_xkey(l16)) << 4));
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int mb = 0; mb < 8; ++mb) {
          if (s == 0)
            mfma16_y_first(acc[mb], rtf[0][mb], xb[0]);
          else
            mfma16_y(acc[mb], rtf[s][mb], xb[s]);
        }
      mfma16_result_fence(acc);
    }
    const int token = tile * T + wave * 16 + l16;
    const bool valid = token < n;
    float s1 = 0.f;
#pragma unroll
    for (int mb = 0; mb < 8; ++mb)
#pragma unroll
      for (int r = 0; r < 4; ++r) s1 += acc[mb][r];
    const float mu = quarter_sum_all(s1) * inv_d;
    float s2 = 0.f, s3 = 0.f, s4 = 0.f;
#pragma unroll
    for (int mb = 0; mb < 8; ++mb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float c = acc[mb][r] - mu;
        acc[mb][r] = c;
        const float c2 = c * c;
        s2 += c2;
        s3 = fmaf(c2, c, s3);
        s4 = fmaf(c2, c2, s4);
      }
    const float m2 = quarter_sum_all(s2) * inv_d, m3 = quarter_sum_all(s3) * inv_d, m4 = quarter_sum_all(s4) * inv_d;
    const bool ok = valid && m2 > 1e-10f * (m2 + mu * mu);  // same rule as finalize_rows_kernel
    // branch-free: a degenerate or out-of-range token gets kappa = 0 and no gradient
    const float m2s = ok ? m2 : 1.f;
    const float inv_m2sq = 1.0f / (m2s * m2s);
    const float kappa = ok ? m4 * inv_m2sq : 0.f;
    float sgn = 1.f, term = kappa;
    if (kappa_target != 0.f) {  // uniform
      const float dk = kappa - kappa_target;
      sgn = (float)((dk > 0.f) - (dk < 0.f));
      term = fabsf(dk);
    }
    const float alpha = ok ? sgn * grad_scale * inv_m2sq : 0.f;
    const float beta = kappa * m2;
    loss_acc += (q == 0 && valid) ? (double)term : 0.0;
    if (want_grad) {
      char* grow = lds + kF128GOff + gbuf * BUF + (wave * 16 + l16) * 256;
#pragma unroll
      for (int mb = 0; mb < 8; ++mb) {
        typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
        bf16x4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float c = acc[mb][r];
          v[r] = (__bf16)(alpha * fmaf(c, fmaf(c, c, -beta), -m3));
        }
        *reinterpret_cast<bf16x4*>(grow + (((4 * mb + q) ^ f128_gkey(l16)) << 3)) = v;  // 8-byte unit: features 4 u .. 4 u + 3
      }
    }
    if (row_kurt && q == 0 && valid) row_kurt[(int64_t)b * n + token] = kappa;
  };

  // E: dR += X^T G of a tile
  auto stage_e = [&](int xbuf, int gbuf) __attribute__((always_inline)) {
    asm volatile("" : "+v"(xa), "+v"(ga));  // (the addresses of the blocks are made here and not kept across the phases)
    const int x0 = xa + xbuf * BUF, g0 = ga + gbuf * BUF;
    intx4 fx[2][2], fg[2][4];
    // operand k of K step s (two transposing reads): the G blocks 0 .. 3, the X blocks 4, 5
    auto fread = [&](auto s_c, auto k_c) __attribute__((always_inline)) {
      constexpr int s = decltype(s_c)::value, k = decltype(k_c)::value;
      const int at = (k < 4 ? g0 : x0) ^ ((k & 3) * kBlock);
      (k < 4 ? fg[s & 1][k & 3] : fx[s & 1][k & 1]) = read_tr_operand(lds, at + s * 32 * 256, (at ^ kRow4) + s * 32 * 256);
    };
    static_for<6>([&](auto k_c) __attribute__((always_inline)) { fread(integral_constant<int, 0>{}, k_c); });
    static_for<32>([&](auto g_c) __attribute__((always_inline)) {
      constexpr int g = decltype(g_c)::value, s = g >> 3, k = g & 7, ib = k >> 2, jb = k & 3;
      __builtin_amdgcn_sched_barrier(0);
      mfma16_dr(acc2[ib][jb], fx[s & 1][ib], fg[s & 1][jb]);
      if constexpr (s + 1 < 4 && k < 6) fread(integral_constant<int, s + 1>{}, integral_constant<int, k>{});
      __builtin_amdgcn_sched_barrier(0);
    });
    mfma16_result_fence(acc2);
  };

  // phase i
  const bool e_first = wave >= 4;
  int xbuf = 0;  // i % 3
  for (int i = 0; i <= my_tiles; ++i) {
    const int xnext = xbuf == 2 ? 0 : xbuf + 1, xprev = xbuf == 0 ? 2 : xbuf - 1;
    const bool with_e = want_grad && i > 0;
    // this wave's rows of X(i) have landed (and with the barrier at the end of this phase everybody's)
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    if (i + 1 < my_tiles) load_tile(wg + (i + 1) * S, xnext);  // buffer last read by E(i-2)
    if (e_first && with_e) stage_e(xprev, (i - 1) & 1);
    if (i < my_tiles) stage_bcd(wg + i * S, xbuf, i & 1);
    if (!e_first && with_e) stage_e(xprev, (i - 1) & 1);
    lds_barrier();  // G(i) is complete, X(i) has landed, the buffers of tile i - 1 are free
    xbuf = xnext;
  }

  // ---- wrap-up: partial dR and partial loss of this workgroup ----------------------------
  if (want_grad) {
    float* out = dR_part + ((int64_t)wg * batch + b) * (D * D);
#pragma unroll
    for (int ib = 0; ib < 2; ++ib)
#pragma unroll
      for (int jb = 0; jb < 4; ++jb)
#pragma unroll
        for (int r = 0; r < 4; ++r) out[(wm4 * 32 + ib * 16 + 4 * q + r) * D + wn2 * 64 + jb * 16 + l16] = acc2[ib][jb][r];
  }
  double* sh = reinterpret_cast<double*>(lds);
  sh[tid] = loss_acc;
  __syncthreads();
#pragma unroll
  for (int s = 256; s >= 1; s >>= 1) {
    if (tid < s) sh[tid] += sh[tid + s];
    __syncthreads();
  }
  if (tid == 0) loss_part[(int64_t)b * S + wg] = sh[0];
}

// ---- single-pass rotate + int4 fake-quant for d = 128 (bf16) -------------------------------
// The four lanes l, l + 16, l + 32, l + 48 hold a whole rotated token row, so the row maximum, the scale, the codes and the
// error sums all come out of ONE pass over X (the generic path parks the rotated rows in an fp32
// staging buffer between the GEMM and a row kernel).
// R is staged in the kernel (stage_rotation; a launch that wrote R^T first was 5 of 101 us of 256 problems and 3 of 11 of a small call).  From there
// every wave is on its own: 16-token tiles, its rows staged through 4 KiB of private LDS (loads of
// the next tile in flight), R^T fragments in accumulation registers, no workgroup barrier.
// 16 x 16 blocks (one token, 32 features per lane) keep a wave under 256 registers, so that two share a SIMD: one wave's
// loads, matrix instructions and quantiser arithmetic hide behind the other's.  256 problems x 4096 tokens: one wave per
// SIMD (32-token tiles, 324 registers, twice the workgroups) 139 us, this form 106 us; two tiles in flight instead of one: 7 % slower.
// Arithmetic identical to the generic path: s = (clip amax) / 7, q = clamp(rint(y (1/s)), -7, 7).
// grid = (waves / 4, batch).
__global__ __launch_bounds__(256, 2) void quant_d128_kernel(const __bf16* __restrict__ X, int64_t ldx,
                                                         int64_t x_batch_stride, const void* __restrict__ R, int64_t ldr, int r_bf16,
                                                         int n, float clip, const float* __restrict__ scales_in,
                                                         float* __restrict__ scales_out, int8_t* __restrict__ codes,
                                                         float2* __restrict__ err) {
  __shared__ __align__(16) char lds_all[128 * 256];  // R first, then 4 KiB a wave
  constexpr int D = 128;
  const int b = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int q = lane >> 4, l16 = lane & 15;
  char* lds = lds_all + wave * (16 * 256);
  X += (int64_t)b * x_batch_stride;
  R = static_cast<const char*>(R) + (int64_t)b * D * ldr * (r_bf16 ? 2 : 4);
  const int tiles = (n + 15) / 16;
  const int wave_id = blockIdx.x * 4 + wave, stride = gridDim.x * 4;

  // chunk i of a lane: tile row q + 4 i, 16-byte column l16
  intx4 nxt[4];
  auto request = [&](int tile) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = tile * 16 + q + 4 * i;
      intx4 v = {0, 0, 0, 0};
      if (tile < tiles && row < n) v = *reinterpret_cast<const intx4*>(X + (int64_t)row * ldx + l16 * 8);
      nxt[i] = v;
    }
  };
  request(wave_id);
  // R^T fragments (K step, block of 16 features) from R, rounded and staged by the workgroup, into accumulation registers
  stage_rotation<256>(R, ldr, r_bf16, lds_all);
  lds_barrier();
  intx4 rtf[4][8];
  const int tr_row = 8 * q + (l16 >> 2), ra = tr_row * 256 + ((((l16 & 3) >> 1) ^ f128_xkey(tr_row)) << 4) + ((l16 & 1) << 3);
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int mb = 0; mb < 8; ++mb) {
      const int at = ra ^ (mb * 32);
      rtf[s][mb] = read_tr_operand(lds_all, at + s * 32 * 256, (at ^ (4 * 256 + 16)) + s * 32 * 256);
    }
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int mb = 0; mb < 8; ++mb) asm volatile("" : "+a"(rtf[s][mb]));
  lds_barrier();  // everybody has its fragments: the room is the waves' own
  for (int tile = wave_id; tile < tiles; tile += stride) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the previous tile's fragment reads are done
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = q + 4 * i;
      *reinterpret_cast<intx4*>(lds + row * 256 + ((l16 ^ f128_xkey(row)) << 4)) = nxt[i];
    }
    request(tile + stride);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // LDS of one wave executes in order; keep the compiler in order too
    floatx4 acc[8];  // features 16 mb + 4 q + r of token l16
    {
      const char* xrow = lds + l16 * 256;
      intx4 xb[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) xb[s] = *reinterpret_cast<const intx4*>(xrow + (((4 * s + q) ^ f128_xkey(l16)) << 4));
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int mb = 0; mb < 8; ++mb) {
          if (s == 0)
            mfma16_y_first(acc[mb], rtf[0][mb], xb[0]);
          else
            mfma16_y(acc[mb], rtf[s][mb], xb[s]);
        }
      mfma16_result_fence(acc);
    }
    const int token = tile * 16 + l16;
    const bool tv = token < n;
    const int64_t to = (int64_t)b * n + token;
    float s;
    if (scales_in) {
      s = tv ? scales_in[to] : 0.f;
    } else {
      float a = 0.f;
#pragma unroll
      for (int mb = 0; mb < 8; ++mb)
#pragma unroll
        for (int r = 0; r < 4; ++r) a = fmaxf(a, fabsf(acc[mb][r]));
      float o = a;
      swap_halves(a, o);
      a = fmaxf(a, o);
      o = a;
      swap_quarters(a, o);
      a = fmaxf(a, o);
      s = __fdiv_rn(__fmul_rn(clip, a), 7.0f);
    }
    if (scales_out && tv && q == 0) scales_out[to] = s;
    if (codes || err) {
      const bool live = s > 0.f;
      const float rinv = live ? __fdiv_rn(1.0f, s) : 0.f;
      const float top = live ? 7.f : 0.f;  // a row with scale 0 gets codes 0
      float e2 = 0.f, y2 = 0.f;
      int8_t* crow = codes + to * D;
#pragma unroll
      for (int m4 = 0; m4 < 2; ++m4) {
        float pk[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          unsigned t[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            // clamp(rint(v)) = rint(clamp(v)) for whole bounds; 1.5 2^23 + v has rint(v) (ties to even) in its low bits
            const float y = acc[4 * m4 + i][e];
            const float v = __builtin_amdgcn_fmed3f(__fmul_rn(y, rinv), -top, top);
            const float m = __fadd_rn(v, 12582912.f);
            t[e] = __float_as_uint(m);
            const float diff = fmaf(-__fsub_rn(m, 12582912.f), s, y);
            e2 = fmaf(diff, diff, e2);
            y2 = fmaf(y, y, y2);
          }
          const unsigned lo = __builtin_amdgcn_perm(t[1], t[0], 0x0c0c0400u), hi = __builtin_amdgcn_perm(t[3], t[2], 0x04000c0cu);
          pk[i] = __uint_as_float(lo | hi);
        }
        // word i of quarter c = features 16 i + 4 c .. + 3 of these 64: transposed among the four lanes of the token,
        // quarter c holds all 16 bytes of block c
        swap_halves(pk[0], pk[2]);
        swap_halves(pk[1], pk[3]);
        swap_quarters(pk[0], pk[1]);
        swap_quarters(pk[2], pk[3]);
        const uintx4 out = {__float_as_uint(pk[0]), __float_as_uint(pk[1]), __float_as_uint(pk[2]), __float_as_uint(pk[3])};
        if (codes && tv) *reinterpret_cast<uintx4*>(crow + 64 * m4 + 16 * q) = out;
      }
      if (err) {
        e2 = quarter_sum_all(e2);
        y2 = quarter_sum_all(y2);
        if (q == 0 && tv) err[to] = make_float2(e2, y2);
      }
    }
  }
}

}  // namespace kt
