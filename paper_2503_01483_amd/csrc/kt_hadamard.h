// kt_hadamard.h -- the online rotations of "Placement of the Rotations" (R3, R4, R5: random
// Hadamard matrices applied to activations at run time):  y = (x * signs) H_d / sqrt(d) per token
// row.  hadamard_rows_kernel: H_d the Sylvester-Hadamard matrix, d = 2^k <= 4096.
// hadamard_cross_kernel: the second factor of H_d = H_m (x) S_{2^k} for the sizes m 2^k that are not
// powers of two (or exceed 4096).  hadamard_onepass_kernel (end of file): both factors in one pass
// over bf16 rows of up to 32768.
//
// HBM-bound: 2 d element reads + 2 d element writes per row against d log2 d additions.  One WAVE
// owns a chunk of 4096 consecutive elements (4096 / d whole rows) and never meets the other waves:
//   1. coalesced 16-byte global loads (issued one chunk ahead) -> fp32 -> its private LDS
//      region (linear order)
//   2. each lane takes 64 consecutive elements: six butterfly stages in registers
//   3. through LDS again, transposed: each lane now holds the elements 64 apart, i.e. the
//      remaining log2(d) - 6 index bits of a row: the last stages in registers
//   4. through LDS back to linear order -> scale, round, coalesced 16-byte stores
// The LDS region is padded by 4 floats per 64 (index i lives at i + 4 (i >> 6)): the 16-byte
// accesses of steps 1, 2, 4 stay aligned and conflict-free (16 lanes of one cycle land 4 or 8
// floats apart modulo the padding), and the 4-byte transposed accesses of step 3 are consecutive
// across lanes.  LDS instructions of one wave execute in order, so no barrier is needed; the
// compiler is kept from reordering them with memory clobbers.
#pragma once
#include "kt_aux.h"
#include "kt_fused_d128.h"  // read_tr_operand

namespace kt {

constexpr int kHadChunk = 4096;
constexpr int kHadRegion = kHadChunk + 4 * (kHadChunk / 64);  // floats per wave

__device__ __forceinline__ void had_lds_fence() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

template <int N>
__device__ __forceinline__ void had_butterflies(float (&a)[64], int first_stage_bit) {
  // N stages on index bits first_stage_bit .. first_stage_bit + N - 1 of the 64 registers
#pragma unroll
  for (int s = 0; s < N; ++s) {
    const int h = 1 << (first_stage_bit + s);
#pragma unroll
    for (int e = 0; e < 64; ++e) {
      if ((e & h) == 0) {
        const float u = a[e], v = a[e | h];
        a[e] = u + v;
        a[e | h] = u - v;
      }
    }
  }
}

// T = float or __bf16; LOG2D in 7..12.  grid.x workgroups of 4 waves walk the chunks.
// sign_rows > 1: the rows are segments of longer rows (sign_rows segments each) and row r takes its
// signs from signs[(r % sign_rows) * D ...].
template <typename T, int LOG2D>
__global__ __launch_bounds__(256) void hadamard_rows_kernel(const T* __restrict__ X, int64_t ldx,
                                                            T* __restrict__ Y, int64_t ldy,
                                                            const int8_t* __restrict__ signs, int64_t n,
                                                            float scale, int sign_rows) {
  constexpr int D = 1 << LOG2D, ROWS = kHadChunk / D, M = LOG2D - 6, VEC = 16 / (int)sizeof(T);
  constexpr int NLD = kHadChunk / (64 * VEC);  // 16-byte accesses per lane and chunk
  extern __shared__ __align__(16) float lds_all[];  // 4 * kHadRegion floats
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float* lds = lds_all + wave * kHadRegion;
  const int64_t chunks = (n + ROWS - 1) / ROWS;
  // the loads of the next chunk are in flight while this one is transformed
  intx4 nxt[NLD];
  auto request = [&](int64_t chunk) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < NLD; ++t) {
      const int i = (t * 64 + lane) * VEC;
      const int64_t row = chunk * ROWS + (i >> LOG2D);
      intx4 r = {0, 0, 0, 0};
      if (chunk < chunks && row < n) r = *reinterpret_cast<const intx4*>(X + row * ldx + (i & (D - 1)));
      nxt[t] = r;
    }
  };
  const int64_t stride = (int64_t)gridDim.x * 4;
  request((int64_t)blockIdx.x * 4 + wave);
  for (int64_t chunk = (int64_t)blockIdx.x * 4 + wave; chunk < chunks; chunk += stride) {
    const int64_t row0 = chunk * ROWS;
    intx4 cur[NLD];
#pragma unroll
    for (int t = 0; t < NLD; ++t) cur[t] = nxt[t];
    request(chunk + stride);
    // 1. registers -> LDS (linear, padded)
#pragma unroll
    for (int t = 0; t < NLD; ++t) {
      const int i = (t * 64 + lane) * VEC;
      const int64_t row = row0 + (i >> LOG2D);
      const int col = i & (D - 1);
      float v[VEC];
      if (row < n) {
        const intx4 raw = cur[t];
        if constexpr (sizeof(T) == 4) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = __int_as_float(raw[e]);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) {  // bf16 -> fp32: the 16 bits are the high half
            v[2 * e] = __int_as_float(raw[e] << 16);
            v[2 * e + 1] = __int_as_float(raw[e] & 0xffff0000);
          }
        }
        if (signs) {
          const int8_t* sg = signs + col;
          if (sign_rows > 1) sg += (int64_t)((unsigned)row % (unsigned)sign_rows) * D;  // rows < 2^31 here
#pragma unroll
          for (int e = 0; e < VEC; ++e) v[e] *= (float)sg[e];
        }
      } else {
#pragma unroll
        for (int e = 0; e < VEC; ++e) v[e] = 0.f;
      }
      float* dst = lds + i + 4 * (i >> 6);
#pragma unroll
      for (int e = 0; e < VEC; e += 4) *reinterpret_cast<floatx4*>(dst + e) = floatx4{v[e], v[e + 1], v[e + 2], v[e + 3]};
    }
    had_lds_fence();
    // 2. 64 consecutive elements per lane (index bits 0..5)
    float a[64];
#pragma unroll
    for (int g = 0; g < 16; ++g) {
      const floatx4 q = *reinterpret_cast<const floatx4*>(lds + 68 * lane + 4 * g);
      a[4 * g] = q[0]; a[4 * g + 1] = q[1]; a[4 * g + 2] = q[2]; a[4 * g + 3] = q[3];
    }
    had_butterflies<6>(a, 0);
    had_lds_fence();
#pragma unroll
    for (int g = 0; g < 16; ++g)
      *reinterpret_cast<floatx4*>(lds + 68 * lane + 4 * g) = floatx4{a[4 * g], a[4 * g + 1], a[4 * g + 2], a[4 * g + 3]};
    had_lds_fence();
    // 3. elements lane + 64 j: index bits 6.. of the chunk; the low M bits of j belong to the row
#pragma unroll
    for (int j = 0; j < 64; ++j) a[j] = lds[lane + 68 * j];
    had_butterflies<M>(a, 0);
    had_lds_fence();
#pragma unroll
    for (int j = 0; j < 64; ++j) lds[lane + 68 * j] = a[j] * scale;
    had_lds_fence();
    // 4. LDS (linear) -> global
#pragma unroll
    for (int t = 0; t < NLD; ++t) {
      const int i = (t * 64 + lane) * VEC;
      const int64_t row = row0 + (i >> LOG2D);
      const int col = i & (D - 1);
      const float* src = lds + i + 4 * (i >> 6);
      float v[VEC];
#pragma unroll
      for (int e = 0; e < VEC; e += 4) {
        const floatx4 q = *reinterpret_cast<const floatx4*>(src + e);
        v[e] = q[0]; v[e + 1] = q[1]; v[e + 2] = q[2]; v[e + 3] = q[3];
      }
      if (row < n) {
        if constexpr (sizeof(T) == 4) {
          *reinterpret_cast<floatx4*>(Y + row * ldy + col) = floatx4{v[0], v[1], v[2], v[3]};
        } else {
          typedef __bf16 bf16x8v __attribute__((ext_vector_type(8)));
          bf16x8v o;
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = (__bf16)v[e];
          *reinterpret_cast<bf16x8v*>(Y + row * ldy + col) = o;
        }
      }
    }
    had_lds_fence();
  }
}

// ---- H_d = H_m (x) S_p2 for d = m p2 --------------------------------------------------------------
// hadamard_rows_kernel has already transformed (and scaled) each of the m segments of p2
// consecutive elements of a row; this kernel mixes the segments, in place:
//   y[a p2 + b] = sum_a' x[a' p2 + b] H_m[a'][a].
// H_m (kind 0: Sylvester; 1: Paley's first construction, q = m - 1; 2: Paley's second, q = m/2 - 1)
// is written into LDS as floats by every workgroup from the quadratic residues of q.  A workgroup
// then walks tiles of 128 columns b of one row: the m x 128 values go through LDS as fp32 (all
// loads before any store, so the transform is in place); a thread owns two columns and four
// outputs a at a time, a wave reads its four H_m columns with one broadcast 16-byte LDS read per a'.
// m is a multiple of 4, p2 a multiple of 128.  LDS: (m*m + 128*CG*m) floats + q bytes.
template <typename T>
__global__ __launch_bounds__(256) void hadamard_cross_kernel(T* __restrict__ Y, int64_t ldy, int64_t n, int m,
                                                             int p2, int kind) {
  extern __shared__ __align__(16) float cross_lds[];
  float* S = cross_lds;
  float* xt = cross_lds + m * m;
  const int quads = m >> 2;
  int CG = quads >= 3 ? 1 : (quads == 2 ? 2 : 4);  // column groups of a tile, see below
  while (CG > 1 && (p2 >> 7) < CG) CG >>= 1;
  unsigned char* isq = reinterpret_cast<unsigned char*>(xt + 128 * CG * m);
  const int tid = threadIdx.x;
  const int h = kind == 2 ? m / 2 : m;  // order of the conference matrix
  const int q = h - 1;
  if (kind != 0) {
    for (int t = tid; t < q; t += 256) isq[t] = 0;
    __syncthreads();
    for (int t = 1 + tid; t < q; t += 256) isq[(t * t) % q] = 1;  // equal values: no race that matters
    __syncthreads();
  }
  for (int idx = tid; idx < m * m; idx += 256) {
    const int i = idx / m, j = idx - i * m;
    float e;
    if (kind == 0) {
      e = (__builtin_popcount(i & j) & 1) ? -1.f : 1.f;
    } else {
      const int u = i % h, v = j % h;
      // conference matrix entry: 0 on the diagonal, border +1 (first column of Paley I: -1),
      // inside the quadratic character of u - v
      float c;
      if (u == v) {
        c = 0.f;
      } else if (u == 0 || v == 0) {
        c = (kind == 1 && v == 0) ? -1.f : 1.f;
      } else {
        int x = (u - v) % q;
        if (x < 0) x += q;
        c = isq[x] ? 1.f : -1.f;
      }
      const float id = u == v ? 1.f : 0.f;
      if (kind == 1) e = c + id;
      else if (i < h && j < h) e = c + id;
      else if (i >= h && j >= h) e = -c - id;
      else e = c - id;
    }
    S[idx] = e;
  }
  __syncthreads();

  // A wave works on 128 columns (two per lane) and four outputs a at a time.  With fewer than four
  // such quads (m < 16) the waves share them out over CG = 2 or 4 column groups of a wider tile.
  const int c2 = tid & 63, g = tid >> 6;
  const int tcols = 128 * CG, ncb = p2 / tcols;
  const int cg = g % CG, q0 = g / CG, qstep = 4 / CG;
  const int64_t tiles = n * ncb;
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int64_t row = tile / ncb;
    const int cb = (int)(tile - row * ncb);
    T* base = Y + row * ldy + (int64_t)cb * tcols + 2 * c2;
    for (int idx = g; idx < m * CG; idx += 4) {
      const int a = idx / CG, k = idx - a * CG;
      float x0, x1;
      if constexpr (sizeof(T) == 4) {
        const float2 v = *reinterpret_cast<const float2*>(base + (int64_t)a * p2 + 128 * k);
        x0 = v.x; x1 = v.y;
      } else {
        const unsigned v = *reinterpret_cast<const unsigned*>(base + (int64_t)a * p2 + 128 * k);
        x0 = __uint_as_float(v << 16); x1 = __uint_as_float(v & 0xffff0000u);
      }
      *reinterpret_cast<float2*>(xt + a * tcols + 128 * k + 2 * c2) = make_float2(x0, x1);
    }
    __syncthreads();
    for (int qd = q0; qd < quads; qd += qstep) {
      float acc[4][2] = {{0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}};
#pragma unroll 4
      for (int a = 0; a < m; ++a) {
        const float2 xv = *reinterpret_cast<const float2*>(xt + a * tcols + 128 * cg + 2 * c2);
        const floatx4 sv = *reinterpret_cast<const floatx4*>(S + a * m + 4 * qd);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          acc[j][0] = fmaf(sv[j], xv.x, acc[j][0]);
          acc[j][1] = fmaf(sv[j], xv.y, acc[j][1]);
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        T* dst = base + (int64_t)(4 * qd + j) * p2 + 128 * cg;
        if constexpr (sizeof(T) == 4) {
          *reinterpret_cast<float2*>(dst) = make_float2(acc[j][0], acc[j][1]);
        } else {
          typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
          bf16x2v o = {(__bf16)acc[j][0], (__bf16)acc[j][1]};
          *reinterpret_cast<bf16x2v*>(dst) = o;
        }
      }
    }
    __syncthreads();
  }
}

// The same factor for bf16 rows on the matrix cores: entries +-1 and bf16 inputs make every product
// exact, the sums run in fp32 as in the vector version.  Per tile of 128 NBW columns of one row
// (NBW = 2^lognb blocks of 32 columns per wave, chosen so that a tile holds about 128 x 128 values):
//   Y_tile^T[c][a] = sum_a' x[a'][c] H_m[a'][a]   =   A (M = c, K = a') times B (K = a', N = a)
// H_m^T sits in LDS as bf16, K-minor, zero-padded to 32-row blocks and 16-wide K steps, and is
// read as ordinary 16-byte fragments (the B operand).  The x tile sits in LDS as loaded (row a' =
// the tile's columns); its fragments (8 consecutive a' of one column per lane, the A operand) come
// from the transposing read ds_read_b64_tr_b16.  Rows a' >= m of the tile are zero and never
// written.  In the accumulators a lane then owns ONE output a and 4 x 4 consecutive columns, so the
// results go to the y tile in LDS with 8-byte stores (rows padded by 16 bytes against bank
// conflicts) and from there to memory as whole row pieces; the loads of the next tile are in
// flight while a tile is worked on.  m NBW <= 128.
// LDS bytes: 32 MB * 32 KS (H) + 16 KS * 256 NBW (x tile) + 32 MB * (256 NBW + 16) (y tile).
__global__ __launch_bounds__(256) void hadamard_cross_mfma_kernel(__bf16* __restrict__ Y, int64_t ldy, int64_t n,
                                                                  int m, int p2, int kind, int lognb) {
  extern __shared__ __align__(16) char cross_raw[];
  const int MB = (m + 31) >> 5, KS = (m + 15) >> 4;
  const int NBW = 1 << lognb, rowb = 256 << lognb, tcols = 128 << lognb;
  const int a_stride = 32 * KS;  // bytes per row of A: 16 KS bf16
  char* A = cross_raw;
  char* xt = A + 32 * MB * a_stride;
  char* yt = xt + 16 * KS * rowb;
  const int rowy = rowb + 16;  // bytes per row of the y tile
  unsigned char* isq = reinterpret_cast<unsigned char*>(yt);  // scratch during set-up only
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int half = lane >> 5, l32 = lane & 31;
  const int h = kind == 2 ? m / 2 : m;
  const int q = h - 1;
  if (kind != 0) {
    for (int t = tid; t < q; t += 256) isq[t] = 0;
    __syncthreads();
    for (int t = 1 + tid; t < q; t += 256) isq[(t * t) % q] = 1;
    __syncthreads();
  }
  // A[a][k] = H_m[k][a] (0 in the padding)
  for (int idx = tid; idx < 32 * MB * 16 * KS; idx += 256) {
    const int a = idx / (16 * KS), k = idx - a * (16 * KS);
    float e = 0.f;
    if (a < m && k < m) {
      const int i = k, j = a;  // entry H_m[i][j]
      if (kind == 0) {
        e = (__builtin_popcount(i & j) & 1) ? -1.f : 1.f;
      } else {
        const int u = i % h, v = j % h;
        float c;
        if (u == v) {
          c = 0.f;
        } else if (u == 0 || v == 0) {
          c = (kind == 1 && v == 0) ? -1.f : 1.f;
        } else {
          int x = (u - v) % q;
          if (x < 0) x += q;
          c = isq[x] ? 1.f : -1.f;
        }
        const float id = u == v ? 1.f : 0.f;
        if (kind == 1) e = c + id;
        else if (i < h && j < h) e = c + id;
        else if (i >= h && j >= h) e = -c - id;
        else e = c - id;
      }
    }
    reinterpret_cast<__bf16*>(A)[idx] = (__bf16)e;
  }
  __syncthreads();  // isq (inside yt) is free again
  for (int i = tid; i < KS * rowb; i += 256) reinterpret_cast<intx4*>(xt)[i] = intx4{0, 0, 0, 0};
  __syncthreads();

  // lane constants of the transposing reads: columns tr_col .. +3 of a 32-column block, row 16 s + tr_row (+4)
  const int g16 = lane >> 4, rr = lane & 15;
  const int tr_col = 16 * (g16 & 1) + 4 * (rr & 3);
  const int tr_row = 8 * (g16 >> 1) + (rr >> 2);
  const int ncb = p2 / tcols;
  const int64_t tiles = n * ncb;
  // tile movement: 16-byte chunk c = tid + 256 i of the tile: row a = c / (16 NBW), chunk c % (16 NBW)
  const int chunk_shift = 4 + lognb, chunk_mask = (16 << lognb) - 1;
  intx4 nxt[8];
  auto request = [&](int64_t tile) __attribute__((always_inline)) {
    const int64_t row = tile / ncb;
    const int cb = (int)(tile - row * ncb);
    const __bf16* src = Y + row * ldy + (int64_t)cb * tcols;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int c = tid + 256 * i, a = c >> chunk_shift;
      if (tile < tiles && a < m) nxt[i] = *reinterpret_cast<const intx4*>(src + (int64_t)a * p2 + (c & chunk_mask) * 8);
    }
  };
  request(blockIdx.x);
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int64_t row = tile / ncb;
    const int cb = (int)(tile - row * ncb);
    __bf16* base = Y + row * ldy + (int64_t)cb * tcols;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int c = tid + 256 * i, a = c >> chunk_shift;
      if (a < m) *reinterpret_cast<intx4*>(xt + a * rowb + (c & chunk_mask) * 16) = nxt[i];
    }
    request(tile + gridDim.x);
    __syncthreads();
    for (int nb = 0; nb < NBW; ++nb) {
      const int col0 = (wave * NBW + nb) * 32;  // this wave's block of 32 columns
      const int tr_lo = tr_row * rowb + (col0 + tr_col) * 2, tr_hi = tr_lo + 4 * rowb;
      floatx16 acc[4];
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[mb][r] = 0.f;
      for (int s = 0; s < KS; ++s) {
        const intx4 bf = read_tr_operand(xt, tr_lo + s * 16 * rowb, tr_hi + s * 16 * rowb);
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
          if (mb < MB) {
            const intx4 af = *reinterpret_cast<const intx4*>(A + (32 * mb + l32) * a_stride + (2 * s + half) * 16);
            acc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, bf),
                                                              __builtin_bit_cast(bf16x8, af), acc[mb], 0, 0, 0);
          }
      }
      // lane: output a = 32 mb + l32, columns col0 + 8 (r / 4) + 4 half + (r & 3)
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
        if (mb < MB) {
          const int a = 32 * mb + l32;
          if (a < m) {
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) {
              typedef __bf16 bf16x4v __attribute__((ext_vector_type(4)));
              const bf16x4v o = {(__bf16)acc[mb][4 * rg], (__bf16)acc[mb][4 * rg + 1], (__bf16)acc[mb][4 * rg + 2],
                                 (__bf16)acc[mb][4 * rg + 3]};
              *reinterpret_cast<bf16x4v*>(yt + a * rowy + (col0 + 8 * rg + 4 * half) * 2) = o;
            }
          }
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int c = tid + 256 * i, a = c >> chunk_shift;
      if (a < m)
        *reinterpret_cast<intx4*>(base + (int64_t)a * p2 + (c & chunk_mask) * 8) =
            *reinterpret_cast<const intx4*>(yt + a * rowy + (c & chunk_mask) * 16);
    }
    // the next tile's stores to xt come after every wave has passed the barrier above (its reads of
    // xt are done), its stores to yt after the next barrier (the copy-out above is done)
  }
}

// ---- both factors in one pass, bf16 rows of up to 32768 elements ------------------------------------
// Two kernels move a row through memory twice.  Here a workgroup keeps a whole row in LDS:
//   H_m (x) S_p2 = H_M (x) S_P,  M = m 2^j <= 32 waves (4, or 8 above d = 16384), P = p2 / 2^j = 64 or 128,
// (H_M = H_m (x) S_2^j).  The H_M factor comes FIRST, on the matrix cores: the inputs are bf16 and the entries +-1,
// so every product is exact and nothing is rounded between the factors.  The entries go in as +-2^-16 and the final scale
// makes up for it: a sum of 32768 bf16 values fits 32 bits whatever they are, and 2^-16 times the smallest one (2^-133) is
// the smallest fp32 number, so the products stay exact.  A wave takes 32 of the M outputs and all P columns, so that the
// S_P factor is butterflies in its own registers (32 x 32 blocks, a lane owns one output and
// 16 columns of each block: five or more index bits are register bits, the sixth is the wave half).
// Per row: registers -> LDS (with the signs, an XOR of the sign bits that is the same for every row; `signs` that are not all
// +-1 go to hadamard_rows_any_factor), request the next row, matrix instructions (the row read with K = input index as the row of the LDS tile, transposing reads), butterflies,
// bf16 results -> the same LDS, 16-byte stores.  Four barriers a row; the workgroups that share a CU overlap.
// LDS rows are 2 P bytes; 64-byte pieces (reads) and 16-byte chunks (results) are XOR-swizzled with the row.
// Bound: HBM, one read and one write of the rows.  512 MiB of rows, two kernels / this one: d = 14336 491 / 221 us
// (4.9 TB/s; 16 rows, set-up and all: 15.9 / 7.2; the first row is requested ahead of the set-up, which makes a row of H_m per thread: with an
// entry at a time and atomics 16 rows took 8.6, of 13824 21.7 instead of 7.1), 13824 683 / 223, 8192 547 / 215, 5120 528 / 243, 28672 483 / 288 (eight
// waves of 256 registers, one workgroup per CU: its barriers overlap with nothing), 1536 (one wave of four at work) 778 / 513.
struct HadamardFactor {
  unsigned long long squares[2];  // bit x: x is a quadratic residue modulo q
  int m, kind, h, q, log2j;       // H_m as in hadamard_cross_kernel; M = m << log2j
};

// whether H_m[a][b] is -1
__device__ __forceinline__ int hadamard_negative(const HadamardFactor& f, int a, int b) {
  int neg = 0;
  if (f.kind == 0) {
    neg = __builtin_popcount(a & b) & 1;
  } else {
    const int alow = a < f.h, blow = b < f.h;
    const int u = alow ? a : a - f.h, v = blow ? b : b - f.h;
    int plus;  // conference matrix entry + identity (u == v: the identity alone)
    if (u == v) {
      plus = 1;
    } else if (u == 0 || v == 0) {
      plus = !(f.kind == 1 && v == 0);
    } else {
      int x = u - v;
      if (x < 0) x += f.q;
      plus = (int)((f.squares[x >> 6] >> (x & 63)) & 1);
    }
    // kind 2: [C + I, C - I; C - I, -C - I]: the diagonal changes sign off the first block, C in the last one
    if (f.kind == 2) {
      if (!alow && !blow) plus ^= 1;
      else if (alow != blow && u == v) plus ^= 1;
    }
    neg = !plus;
  }
  return neg;
}

// The same for all a at once, bit a.  Off its first row and column the conference matrix is circulant: its row is the first one, rotated.
typedef unsigned __int128 Bits128;
__device__ __forceinline__ Bits128 hadamard_negative_row(const HadamardFactor& f, int b) {
  if (f.kind == 0) {  // m <= 8
    unsigned row = 0u;
    for (int a = 0; a < f.m; ++a) row |= (unsigned)(__builtin_popcount(a & b) & 1) << a;
    return row;
  }
  const Bits128 one = 1, ones_q = (one << f.q) - 1;
  const Bits128 squares = (Bits128)f.squares[1] << 64 | f.squares[0], nonsquares = ones_q & ~squares & ~one;  // (0 is the diagonal)
  const int v = b < f.h ? b : b - f.h;
  Bits128 row;
  if (v == 0) row = f.kind == 1 ? ones_q << 1 : 0;
  else row = ((nonsquares << (v - 1) | nonsquares >> (f.q - (v - 1))) & ones_q) << 1;
  if (f.kind == 2) {
    const Bits128 off = row ^ one << v;
    row = b < f.h ? row | off << f.h : off | (~row & (ones_q << 1 | one)) << f.h;
  }
  return row;
}

// ---- fp32 rows of H_m (x) S_p2 in one pass: a workgroup per row, the row in LDS ------------------------
// The Sylvester factor as in hadamard_rows_kernel (a wave per 4096 elements, the same layout, steps 1 to 3), then H_m straight from
// LDS to memory as in hadamard_cross_kernel; the loads of the next row are in flight meanwhile.  The order of every sum
// is that of the two kernels.  Where it is taken it saves a launch and half the traffic; m products per element on the vector ALU, with
// two workgroups on a CU (the registers of 64 values and of the next row), keep it from HBM's rate (hadamard_f32_lds has the figures).
// Three workgroups a CU spilled 68 registers and lost 20 to 40 %.
// Needs d <= 4096 WAVES and LDS for the row (padded, whole blocks of 4096) and H_m as floats.
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void hadamard_f32_onepass_kernel(const float* X, int64_t ldx, float* Y, int64_t ldy,
                                                                          const int8_t* __restrict__ signs, int64_t n, int d, int p2,
                                                                          int log2p, float scale, HadamardFactor f) {
  constexpr int NT = 64 * WAVES, NLD = 16;  // 16-byte loads per thread for 4096 elements a wave
  extern __shared__ __align__(16) float row_lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), m = f.m;
  const int blocks = (d + kHadChunk - 1) / kHadChunk;
  float* S = row_lds + blocks * kHadRegion;
  for (int i = tid; i < m * m; i += NT) S[i] = hadamard_negative(f, i / m, i % m) ? -1.f : 1.f;
  floatx4 nxt[NLD];
  auto request = [&](int64_t row) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < NLD; ++t) {
      const int i = (t * NT + tid) * 4;
      if (row < n && i < d) nxt[t] = *reinterpret_cast<const floatx4*>(X + row * ldx + i);
    }
  };
  request(blockIdx.x);
#pragma unroll 1
  for (int64_t row = blockIdx.x; row < n; row += gridDim.x) {
#pragma unroll
    for (int t = 0; t < NLD; ++t) {
      const int i = (t * NT + tid) * 4;
      if (i < d) {
        floatx4 v = nxt[t];
        if (signs) {
          const char4 sg = *reinterpret_cast<const char4*>(signs + i);
          v = floatx4{v[0] * (float)sg.x, v[1] * (float)sg.y, v[2] * (float)sg.z, v[3] * (float)sg.w};
        }
        *reinterpret_cast<floatx4*>(row_lds + i + 4 * (i >> 6)) = v;
      }
    }
    __syncthreads();
    request(row + gridDim.x);
    if (wave < blocks) {  // (what lies behind the row in its last block never meets the row: other segments)
      float* lds = row_lds + wave * kHadRegion;
      float a[64];
#pragma unroll
      for (int g = 0; g < 16; ++g) {
        const floatx4 q = *reinterpret_cast<const floatx4*>(lds + 68 * lane + 4 * g);
        a[4 * g] = q[0]; a[4 * g + 1] = q[1]; a[4 * g + 2] = q[2]; a[4 * g + 3] = q[3];
      }
      had_butterflies<6>(a, 0);
      had_lds_fence();
#pragma unroll
      for (int g = 0; g < 16; ++g)
        *reinterpret_cast<floatx4*>(lds + 68 * lane + 4 * g) = floatx4{a[4 * g], a[4 * g + 1], a[4 * g + 2], a[4 * g + 3]};
      had_lds_fence();
#pragma unroll
      for (int j = 0; j < 64; ++j) a[j] = lds[lane + 68 * j];
      static_for<6>([&](auto s_c) __attribute__((always_inline)) {
        constexpr int s = decltype(s_c)::value;
        if (6 + s < log2p) had_butterflies<1>(a, s);
      });
      had_lds_fence();
#pragma unroll
      for (int j = 0; j < 64; ++j) lds[lane + 68 * j] = a[j] * scale;
    }
    __syncthreads();
    // 128 columns of a segment (two per lane) and four outputs at a time
    const int quads = m >> 2, items = (p2 >> 7) * quads;
    for (int item = wave; item < items; item += WAVES) {
      const int g = item / quads, qd = item - g * quads, c = 128 * g + 2 * lane;
      float acc[4][2] = {{0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}};
#pragma unroll 4
      for (int k = 0; k < m; ++k) {
        const int i = k * p2 + c;
        const float2 xv = *reinterpret_cast<const float2*>(row_lds + i + 4 * (i >> 6));
        const floatx4 sv = *reinterpret_cast<const floatx4*>(S + k * m + 4 * qd);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          acc[j][0] = fmaf(sv[j], xv.x, acc[j][0]);
          acc[j][1] = fmaf(sv[j], xv.y, acc[j][1]);
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) *reinterpret_cast<float2*>(Y + row * ldy + (4 * qd + j) * p2 + c) = make_float2(acc[j][0], acc[j][1]);
    }
    __syncthreads();
  }
}

// The rows for `signs` that are not all +-1 (0 to drop a channel, say): a sum of M products per lane, its column, and wave,
// its output, in fp32; the S_P factor across the lanes.  Correct, not fast: x times such a factor is no bf16 number.
template <int LOGP, int WAVES>
__device__ __forceinline__ void hadamard_rows_any_factor(const __bf16* X, int64_t ldx, __bf16* Y, int64_t ldy, const int8_t* signs,
                                                         int64_t n, float scale, const HadamardFactor& fac, char* lds) {
  constexpr int P = 1 << LOGP, CPR = P / 8, NT = 64 * WAVES;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, M = fac.m << fac.log2j;
  const __bf16* tile = reinterpret_cast<const __bf16*>(lds);
#pragma unroll 1
  for (int64_t row = blockIdx.x; row < n; row += gridDim.x) {
#pragma unroll 1
    for (int c = tid; c < M * CPR; c += NT) reinterpret_cast<intx4*>(lds)[c] = *reinterpret_cast<const intx4*>(X + row * ldx + 8 * c);
    __syncthreads();
#pragma unroll 1
    for (int o = wave; o < M; o += WAVES) {
      const int low = o & ((1 << fac.log2j) - 1);
      float u[P / 64] = {};
#pragma unroll 1
      for (int i = 0; i < M; ++i) {
        const bool neg = (hadamard_negative(fac, i >> fac.log2j, o >> fac.log2j) ^ __builtin_popcount(i & low)) & 1;
#pragma unroll
        for (int e = 0; e < P / 64; ++e) {
          const float v = (float)tile[i * P + 64 * e + lane] * 0x1p-16f * (float)signs[i * P + 64 * e + lane];
          u[e] += neg ? -v : v;
        }
      }
      if constexpr (P == 128) {
        const float a = u[0], b = u[1];
        u[0] = a + b;
        u[1] = a - b;
      }
#pragma unroll
      for (int st = 1; st < 64; st <<= 1)
#pragma unroll
        for (int e = 0; e < P / 64; ++e) {
          const float other = __shfl_xor(u[e], st);
          u[e] = lane & st ? other - u[e] : u[e] + other;
        }
#pragma unroll
      for (int e = 0; e < P / 64; ++e) Y[row * ldy + o * P + 64 * e + lane] = (__bf16)(u[e] * scale);
    }
    __syncthreads();
  }
}

// LOGP = log2 P; 64 WAVES threads; d <= 32 WAVES P; scale = 2^16 / sqrt(d)
template <int LOGP, int WAVES>
__global__ __launch_bounds__(64 * WAVES, 2) void hadamard_onepass_kernel(const __bf16* __restrict__ X, int64_t ldx,
                                                                                  __bf16* __restrict__ Y, int64_t ldy,
                                                                                  const int8_t* __restrict__ signs, int64_t n,
                                                                                  float scale, HadamardFactor fac) {
  constexpr int P = 1 << LOGP, NBLK = P / 32, ROWB = 2 * P, CPR = P / 8;  // CPR: 16-byte chunks per tile row
  constexpr int NT = 64 * WAVES, KSM = 2 * WAVES, NCH = 32 * WAVES * CPR / NT;  // matrix steps, chunks per thread: at most
  constexpr bool PACKED = WAVES == 8;  // the matrix operands leave few registers
  extern __shared__ __align__(16) char had_lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5, l32 = lane & 31;
  const int M = fac.m << fac.log2j, KS = (M + 15) >> 4, chunks = M * CPR;
  // 64-byte piece of a row read by a transposing read, and 16-byte chunk of a result row: see above
  auto read_key = [](int k) __attribute__((always_inline)) { return LOGP == 6 ? (k >> 1) & 1 : k & 3; };
  auto out_key = [](int a) __attribute__((always_inline)) { return LOGP == 6 ? (a >> 1) & 7 : a & 15; };

  unsigned sg[NCH][2];  // requested first, looked at behind the set-up of the table
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = tid + NT * i;
    sg[i][0] = sg[i][1] = 0x01010101u;
    if (signs && c < chunks) __builtin_memcpy(sg[i], signs + 8 * c, 8);  // (any alignment)
  }
  intx4 nxt[NCH];
  auto request = [&](int64_t row) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = tid + NT * i;
      if (row < n && c < chunks) nxt[i] = *reinterpret_cast<const intx4*>(X + row * ldx + 8 * c);
    }
  };
  if constexpr (!PACKED) request(blockIdx.x);  // (with eight waves the set-up takes all registers)
  // the signs of H_m as 128-bit rows in LDS, bit a of row b; and behind them a word a wave, not zero if its part of `signs` holds anything but +-1
  unsigned* tab = reinterpret_cast<unsigned*>(had_lds);
  if (tid < fac.m) {
    const Bits128 row = hadamard_negative_row(fac, tid);
    *reinterpret_cast<uintx4*>(tab + 4 * tid) = uintx4{(unsigned)row, (unsigned)(row >> 32), (unsigned)(row >> 64), (unsigned)(row >> 96)};
  }
  unsigned other = 0u;  // not zero: this thread has seen a value that is neither 1 nor -1
  unsigned flip8[(NCH + 3) / 4];  // the sign bits of a chunk's eight values, one byte per chunk
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    unsigned byte = 0u;
#pragma unroll
    for (int w = 0; w < 2; ++w) {
      const unsigned neg = sg[i][w] >> 7 & 0x01010101u;
      other |= sg[i][w] ^ (neg * 0xfeu | 0x01010101u);
      byte |= (neg * 0x10204080u >> 28) << (4 * w);  // bits 0, 8, 16, 24 side by side
    }
    flip8[i / 4] = (i % 4 ? flip8[i / 4] : 0u) | byte << (8 * (i % 4));
  }
  const bool wave_other = __any(other != 0u);
  if (lane == 0) tab[4 * fac.m + wave] = wave_other;
  __syncthreads();
  unsigned any_other = 0u;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) any_other |= tab[4 * fac.m + w];
  auto sign_words = [](unsigned byte) __attribute__((always_inline)) {  // the sign bits of eight bf16 values
    intx4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = (int)((byte << (15 - 2 * e) & 0x8000u) | (byte << (30 - 2 * e) & 0x80000000u));
    return v;
  };
  // this wave's 32 columns of H_M as B operands: lane = output o = 32 wave + l32, 8 inputs i = 16 s + 8 half + e;
  // H_M[i][o] = H_m[i / 2^j][o / 2^j] (-1)^(common bits of i and o below 2^j)
  intx4 hf[KSM];
  {
    const int o = 32 * wave + l32, low = o & ((1 << fac.log2j) - 1);
    unsigned row[4] = {0u, 0u, 0u, 0u};
    if (o < M) {
#pragma unroll
      for (int w = 0; w < 4; ++w) row[w] = tab[4 * (o >> fac.log2j) + w];
    }
    // the eight inputs: bits 0 .. 2 of i give one pattern, those above flip all of it
    const unsigned within = (low & 1 ? 0xaau : 0u) ^ (low & 2 ? 0xccu : 0u) ^ (low & 4 ? 0xf0u : 0u);
#pragma unroll
    for (int s = 0; s < KSM; ++s) {
      const int i0 = 16 * s + 8 * half, a0 = i0 >> fac.log2j;
      const unsigned word = a0 < 64 ? (a0 < 32 ? row[0] : row[1]) : (a0 < 96 ? row[2] : row[3]);
      unsigned byte = word >> (a0 & 31);  // the eight inputs share a word: a0 is a multiple of 8 / 2^j, and 2^j of them an entry of H_m
      if (fac.log2j >= 3) byte = byte & 1u ? 0xffu : 0u;
      else if (fac.log2j == 2) byte = (byte & 1u ? 0x0fu : 0u) | (byte & 2u ? 0xf0u : 0u);
      else if (fac.log2j == 1) byte = (byte & 1u) * 0x03u | (byte & 2u) * 0x06u | (byte & 4u) * 0x0cu | (byte & 8u) * 0x18u;
      byte ^= within ^ (__builtin_popcount(i0 & low) & 1 ? 0xffu : 0u);
      const intx4 signs8 = sign_words(byte);
#pragma unroll
      for (int w = 0; w < 4; ++w)  // (M is a multiple of 4; bf16 2^-16 is 0x3780)
        hf[s][w] = i0 + 2 * w < M && o < M ? signs8[w] | 0x37803780 : 0;
      if constexpr (PACKED || LOGP == 6) asm volatile("" : "+v"(hf[s]));  // finished here: half-made words that wait for their end at the loop were spilled
    }
  }
  __syncthreads();  // the table has been read
  if (__builtin_expect(any_other != 0u, 0)) {
    hadamard_rows_any_factor<LOGP, WAVES>(X, ldx, Y, ldy, signs, n, scale, fac, had_lds);
    return;
  }
  // the words to XOR a chunk with (PACKED: made from the byte every time)
  intx4 flip[PACKED ? 1 : NCH];
#pragma unroll
  for (int i = 0; i < (PACKED ? 0 : NCH); ++i) flip[i] = sign_words(flip8[i / 4] >> (8 * (i % 4)) & 0xffu);
  // tile rows M .. 16 KS - 1 meet zeros of H_M: they have to be finite
  for (int c = chunks + tid; c < 16 * KS * CPR; c += NT) reinterpret_cast<intx4*>(had_lds)[c] = intx4{0, 0, 0, 0};

  const int g16 = lane >> 4, rr = lane & 15;
  const int tr_row = 8 * (g16 >> 1) + (rr >> 2), tr_col = 16 * (g16 & 1) + 4 * (rr & 3);
  int tr[NBLK];
#pragma unroll
  for (int b = 0; b < NBLK; ++b) tr[b] = tr_row * ROWB + ((b ^ read_key(tr_row)) << 6) + 2 * tr_col;

  if constexpr (PACKED) request(blockIdx.x);
#pragma unroll 1
  for (int64_t row = blockIdx.x; row < n; row += gridDim.x) {
    if constexpr (PACKED) {  // (or the compiler makes all of the words once and spills them)
#pragma unroll
      for (int i = 0; i < (NCH + 3) / 4; ++i) asm volatile("" : "+v"(flip8[i]));
    }
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = tid + NT * i, k = c / CPR, pos = c % CPR;
      if (c < chunks) *reinterpret_cast<intx4*>(had_lds + k * ROWB + ((pos ^ (read_key(k) << 2)) << 4)) = nxt[i] ^ (PACKED ? sign_words(flip8[i / 4] >> (8 * (i % 4)) & 0xffu) : flip[PACKED ? 0 : i]);
    }
    request(row + gridDim.x);
    lds_barrier();  // (the requested row stays in flight)
    floatx16 acc[NBLK];
#pragma unroll
    for (int b = 0; b < NBLK; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[b][r] = 0.f;
    if (32 * wave < M) {
#pragma unroll
      for (int s = 0; s < KSM; ++s)
        if (s < KS) {
#pragma unroll
          for (int b = 0; b < NBLK; ++b) {
            const intx4 xf = read_tr_operand(had_lds, tr[b] + s * 16 * ROWB, tr[b] + s * 16 * ROWB + 4 * ROWB);
            acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, xf), __builtin_bit_cast(bf16x8, hf[s]),
                                                             acc[b], 0, 0, 0);
          }
          __builtin_amdgcn_sched_barrier(0);  // fragments of one step at a time
        }
    }
    lds_barrier();  // every wave has read the row
    // lane: output 32 wave + l32, column 32 b + 8 (r / 4) + 4 half + (r & 3): index bits 0, 1 (r & 3), 3, 4 (r / 4) and 5 .. (b)
#pragma unroll
    for (int st = 1; st < 16; st <<= 1)
#pragma unroll
      for (int b = 0; b < NBLK; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if ((r & st) == 0) {
            const float u = acc[b][r], v = acc[b][r | st];
            acc[b][r] = u + v;
            acc[b][r | st] = u - v;
          }
#pragma unroll
    for (int st = 1; st < NBLK; st <<= 1)
#pragma unroll
      for (int b = 0; b < NBLK; ++b)
        if ((b & st) == 0) {
          const floatx16 u = acc[b], v = acc[b | st];
          acc[b] = u + v;
          acc[b | st] = u - v;
        }
    // bit 2, the wave half: exchanging registers r / 4 even and odd, the lower half ends up with the eight columns of the
    // even group, the upper half with those of the odd one: 16 bytes of a result row per lane
    const int a = 32 * wave + l32;
    if (a < M) {
#pragma unroll
      for (int b = 0; b < NBLK; ++b)
#pragma unroll
        for (int gp = 0; gp < 2; ++gp) {
          typedef __bf16 bf16x8v __attribute__((ext_vector_type(8)));
          bf16x8v o;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            float x = acc[b][8 * gp + i], y = acc[b][8 * gp + 4 + i];
            swap_halves(x, y);
            o[i] = (__bf16)((x + y) * scale);
            o[4 + i] = (__bf16)((x - y) * scale);
          }
          const int pos = 4 * b + 2 * gp + half;
          *reinterpret_cast<bf16x8v*>(had_lds + a * ROWB + ((pos ^ out_key(a)) << 4)) = o;
        }
    }
    lds_barrier();
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = tid + NT * i, k = c / CPR, pos = c % CPR;
      if (c < chunks)
        *reinterpret_cast<intx4*>(Y + row * ldy + 8 * c) = *reinterpret_cast<const intx4*>(had_lds + k * ROWB + ((pos ^ out_key(k)) << 4));
    }
    lds_barrier();  // the results have been read: the next row may come
  }
}

}  // namespace kt
