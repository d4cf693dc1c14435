// kt_epilogues.h -- what each GEMM on the path does with its accumulator tile.
//
// Every functor is called as epi(acc, batch, tm, tn, ks, m0, n0) once the main
// loop is done; `skip(batch)` lets a launch return early (used by the Cayley
// fixed-point iteration once it has converged).
#pragma once
#include "kt_gemm.h"
#include "kt_gemm32.h"

namespace kt {

template <typename T>
__device__ __forceinline__ T from_float(float v);
template <>
__device__ __forceinline__ float from_float<float>(float v) { return v; }
template <>
__device__ __forceinline__ __bf16 from_float<__bf16>(float v) { return (__bf16)v; }

struct EpiBase {
  static constexpr bool kSwap = false;  // accumulator layout the epilogue takes (Frag)
  __device__ __forceinline__ bool skip(int) const { return false; }
};

// Sums over the four lane quarters of a wave (a column of a 16-row block is spread over them), on the vector ALU:
// v_permlane32_swap exchanges the upper half of its first operand with the lower half of the second,
// v_permlane16_swap the odd quarters of the first with the even ones of the second.
__device__ __forceinline__ void swap_halves(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap_quarters(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}
// the sum of the quarters, in every lane
__device__ __forceinline__ float quarter_sum_all(float x) {
  float y = x;
  swap_halves(x, y);
  x += y;
  y = x;
  swap_quarters(x, y);
  return x + y;
}
struct OpAdd { static __device__ __forceinline__ float of(float a, float b) { return a + b; } };
struct OpMax { static __device__ __forceinline__ float of(float a, float b) { return fmaxf(a, b); } };
// four values v0..v3 per lane, reduced over the quarters: quarter k ends up with the total of v_k
template <class Op>
__device__ __forceinline__ float quarter_reduce4(float v0, float v1, float v2, float v3) {
  swap_halves(v0, v2);
  swap_halves(v1, v3);
  float u0 = Op::of(v0, v2), u1 = Op::of(v1, v3);
  swap_quarters(u0, u1);
  return Op::of(u0, u1);
}
// v_q of the lane's quarter q
__device__ __forceinline__ float quarter_pick(int q, float v0, float v1, float v2, float v3) {
  const float a = (q & 1) ? v1 : v0, b = (q & 1) ? v3 : v2;
  return (q & 2) ? b : a;
}

// A store of 8 or 16 bytes, PAST_L2: in units of 8 that are visible to the whole device once they have completed.
template <bool PAST_L2, class V, class E>
__device__ __forceinline__ void put(E* p, V v) {
  if constexpr (PAST_L2) {
    uint64_t w[sizeof(V) / 8];
    __builtin_memcpy(w, &v, sizeof(V));
#pragma unroll
    for (size_t i = 0; i < sizeof(V) / 8; ++i)
      __hip_atomic_store(reinterpret_cast<uint64_t*>(p) + i, w[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else {
    *reinterpret_cast<V*>(p) = v;
  }
}

// ---- forward pass: per-token moments of y over the hidden dimension ---------------
// m = output feature (reduced in registers), n = token (one per lane).
// part[(batch*P + p)*n_tokens + token] = {mean_p, sum c^2, sum c^3, sum c^4}, c = y - mean_p, over
// the WTM features wave-row p = tm*WGM + wm owns: the mean first, then sums about it (two passes
// over the registers), so that a row whose mean is large against its spread loses nothing to
// cancellation in fp32; the partials of a row are merged in fp64 (row_central_sums in kt_aux.h).
// bf16, 64 features a wave: the two waves of a token merge theirs, so that a partial is 128 features with every tile.
// PAST_L2: for readers in the same launch (kt_rowsync.h), one partial a tile, P = tiles: what they read goes past the L2 as well.
template <class TL, bool PAST_L2 = false>
struct EpiMoments : EpiBase {
  static constexpr bool kMerge = sizeof(typename TL::T) == 2 && TL::WTM == 64;
  static constexpr bool kExchange = PAST_L2 && !kMerge;
  static_assert(TL::MB % 4 == 0 && TL::NB % 4 == 0, "features and tokens are taken 64 at a time");
  floatx4* part;
  int n_tokens, d, P;
  __device__ __forceinline__ void operator()(floatx4 (&acc)[TL::MB][TL::NB], int batch, int tm,
                                             int, int, int m0, int n0) const {
    const Frag<TL> f(thread_id<PAST_L2>());
    const int p = tm * TL::WGM + f.wm;
    int blocks = 0;
#pragma unroll
    for (int mb = 0; mb < TL::MB; ++mb) blocks += (m0 + f.m_block(mb) < d) ? 1 : 0;
    const float inv_cnt = blocks > 0 ? 1.0f / (float)(16 * blocks) : 0.f;
    // 64 tokens (four blocks of columns) at a time: quarter k of the wave ends up with the sums of block k, i.e.
    // lane l with those of token l of the 64
    floatx4 own = {0.f, 0.f, 0.f, 0.f};  // kExchange: of 64-token group wm
#pragma unroll
    for (int g = 0; g < TL::NB / 4; ++g) {
      float mean[4], s2[4], s3[4], s4[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int nb = 4 * g + k;
        float s1 = 0.f;
#pragma unroll
        for (int mb = 0; mb < TL::MB; ++mb) {
          if (m0 + f.m_block(mb) < d) {
#pragma unroll
            for (int r = 0; r < 4; ++r) s1 += acc[mb][nb][r];
          }
        }
        mean[k] = quarter_sum_all(s1) * inv_cnt;
        s2[k] = 0.f; s3[k] = 0.f; s4[k] = 0.f;
#pragma unroll
        for (int mb = 0; mb < TL::MB; ++mb) {
          if (m0 + f.m_block(mb) < d) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float c = acc[mb][nb][r] - mean[k];
              const float c2 = c * c;
              s2[k] += c2;
              s3[k] = fmaf(c2, c, s3[k]);
              s4[k] = fmaf(c2, c2, s4[k]);
            }
          }
        }
      }
      const int token = n0 + f.wn * TL::WTN + 64 * g + f.lane;
      floatx4 v = {quarter_pick(f.q, mean[0], mean[1], mean[2], mean[3]),
                   quarter_reduce4<OpAdd>(s2[0], s2[1], s2[2], s2[3]),
                   quarter_reduce4<OpAdd>(s3[0], s3[1], s3[2], s3[3]),
                   quarter_reduce4<OpAdd>(s4[0], s4[1], s4[2], s4[3])};
      if constexpr (kMerge) {
        static_assert(!kMerge || (TL::BM == 128 && TL::NB == 4), "two waves hold the 128 features of 64 tokens");
        extern __shared__ __align__(16) char lds[];
        floatx4* other = reinterpret_cast<floatx4*>(lds) + 64 * f.wn + f.lane;
        __syncthreads();  // (the last fragments have been read)
        if (f.wm == 1) *other = v;
        __syncthreads();
        if (f.wm == 1) return;
        v = merged(v, *other, 64.0);
      }
      if constexpr (kExchange) {
        static_assert(!kExchange || (TL::WGM == 2 && TL::NB == 8), "two waves hold the features of 128 tokens");
        extern __shared__ __align__(16) char lds[];
        floatx4* sh = reinterpret_cast<floatx4*>(lds) + 64 * (2 * f.wn + g) + f.lane;
        if (g == 0) __syncthreads();  // (the last fragments have been read)
        if (f.wm == g) own = v;
        else *sh = v;
        if (g == 0) continue;
        __syncthreads();
        const floatx4 other = reinterpret_cast<floatx4*>(lds)[64 * (2 * f.wn + f.wm) + f.lane];
        const int mine = n0 + f.wn * TL::WTN + 64 * f.wm + f.lane;
        // the last tile of d % 256 = 128 has nothing in its second half
        v = m0 + TL::WTM < d ? merged(f.wm == 0 ? own : other, f.wm == 0 ? other : own, (double)TL::WTM) : f.wm == 0 ? own : other;
        if (mine < n_tokens) put<PAST_L2>(&part[((int64_t)batch * P + tm) * n_tokens + mine], v);
        return;
      }
      const int pp = kMerge ? tm : p;
      if (token < n_tokens && pp < P) put<PAST_L2>(&part[((int64_t)batch * P + pp) * n_tokens + token], v);
    }
  }
  // two partials of cnt values each as one (the shift formulas of row_central_sums)
  static __device__ __forceinline__ floatx4 merged(const floatx4& a, const floatx4& b, double cnt) {
    const double mu = 0.5 * ((double)a[0] + (double)b[0]);
    double m2 = 0.0, m3 = 0.0, m4 = 0.0;
    auto add = [&](const floatx4& v) __attribute__((always_inline)) {
      const double e = (double)v[0] - mu, e2 = e * e;
      m2 += (double)v[1] + cnt * e2;
      m3 += (double)v[2] + 3.0 * e * (double)v[1] + cnt * e2 * e;
      m4 += (double)v[3] + 4.0 * e * (double)v[2] + 6.0 * e2 * (double)v[1] + cnt * e2 * e2;
    };
    add(a);
    add(b);
    return floatx4{(float)mu, (float)m2, (float)m3, (float)m4};
  }
};

// ---- backward pass: recomputed y -> dL/dy, stored token-minor ---------------------
// coef[token] = {alpha, mu, beta, m3};  g = alpha * (c (c^2 - beta) - m3), c = y - mu.
//
// Layout of GT (dR = X^T G reads X where it lies, its rows taken in this order): rows are
// features, and inside every group of 64 tokens the tokens are PERMUTED,
//     position(t) = (t & 15) * 4 + ((t & 63) >> 4),
// because the contraction over tokens does not care in which order the tokens come as
// long as both operands agree.  In the accumulator layout a lane owns tokens
// t, t+16, t+32, t+48 of a group, so with this order its values for one feature are
// ADJACENT in memory: one 8-byte store per feature instead of four 2-byte ones, and the 16
// lanes of a quarter cover 128 contiguous bytes (256 of the fp32 Y that is kept).  Tokens in
// [n_tokens, ldt) are written as zero so the padded K range contributes nothing; ldt is a
// multiple of 128.
// Rows are stored in blocks of tb tokens (tb a multiple of 128): position p of feature f
// lives at  (p / tb) * d * tb + f * tb + p % tb  (one block, tb = ldt, is the plain layout).

// dL/dy of one entry from the row's coefficients {alpha, mu, beta, m3}; alpha = 0 (padding tokens, rows
// without spread) gives 0 by itself as long as y is finite.  One definition for the recompute epilogue and
// for the kernel that reads a kept Y, so that the two paths round alike.
__device__ __forceinline__ float grad_value(float y, float alpha, float mu, float beta, float m3) {
  const float c = y - mu;
  return alpha * fmaf(c, fmaf(c, c, -beta), -m3);
}

template <class TL>
struct EpiGrad : EpiBase {
  static_assert(TL::MB % 4 == 0 && TL::NB % 4 == 0, "features and tokens are taken 64 at a time");
  using T = typename TL::T;
  const floatx4* coef;
  T* GT;
  int64_t ldt, tb, batch_stride;
  int n_tokens, d;
  __device__ __forceinline__ void operator()(floatx4 (&acc)[TL::MB][TL::NB], int batch, int,
                                             int, int, int m0, int n0) const {
    store(acc, batch, m0, n0, [&](int t) __attribute__((always_inline)) {
      floatx4 c4 = {0.f, 0.f, 0.f, 0.f};  // alpha = 0 zeroes the padding tokens
      if (n0 + t < n_tokens) c4 = coef[(int64_t)batch * n_tokens + n0 + t];
      return c4;
    });
  }
  // coef_of(t): the coefficients of token n0 + t
  template <bool AGAIN = false, class CoefOf>
  __device__ __forceinline__ void store(floatx4 (&acc)[TL::MB][TL::NB], int batch, int m0, int n0, CoefOf coef_of) const {
    typedef T vecT __attribute__((ext_vector_type(4)));
    const Frag<TL> f(thread_id<AGAIN>());
#pragma unroll
    for (int g = 0; g < TL::NB / 4; ++g) {
      const int group0 = n0 + f.wn * TL::WTN + 64 * g;  // the 64-token group
      if (group0 >= ldt) return;
      // the lane's tokens group0 + 16 k + l16 lie at position group0 + 4 l16 + k (a group is in one block): a uniform base and 32 bits a lane
      const int first = __builtin_amdgcn_readfirstlane(group0), blk = first / (int)tb;
      char* base = reinterpret_cast<char*>(GT + (int64_t)batch * batch_stride + (int64_t)blk * d * tb + (first - blk * (int)tb) +
                                           (int64_t)__builtin_amdgcn_readfirstlane(m0 + f.m_block(0)) * tb);
      const uint32_t lane_off = (uint32_t)(4 * f.q * (int)tb + 4 * f.l16) * (uint32_t)sizeof(T);
      float alpha[4], mu[4], beta[4], m3[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const floatx4 c4 = coef_of(group0 - n0 + 16 * k + f.l16);
        alpha[k] = c4[0]; mu[k] = c4[1]; beta[k] = c4[2]; m3[k] = c4[3];
      }
#pragma unroll
      for (int mb = 0; mb < TL::MB; ++mb) {
        if (m0 + f.m_block(mb) < d) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            vecT v;
#pragma unroll
            for (int k = 0; k < 4; ++k)  // (the accumulators of padding tokens come from re-read valid rows and are finite)
              v[k] = from_float<T>(grad_value(acc[mb][4 * g + k][r], alpha[k], mu[k], beta[k], m3[k]));
            *reinterpret_cast<vecT*>(base + (int64_t)((16 * mb + r) * (int)tb) * (int64_t)sizeof(T) + lane_off) = v;
          }
        }
      }
    }
  }
};

// ---- forward pass that also keeps Y = X R ("Learning the Rotations"): the moments of EpiMoments (Eq. 3), and the fp32 accumulators written
// in the layout of GT above (features on the rows, tokens permuted inside groups of 64, blocks of tb
// tokens): one 16-byte store per lane, feature and group, 256 contiguous bytes per feature.  grad_from_y_kernel then turns YT into GT entry by
// entry, which replaces the recompute GEMM of the backward pass (same accumulators, same arithmetic: the
// gradient is bit-identical) at the price of n d 4 bytes of scratch, one write and one read of them.
template <class TL>
struct EpiMomentsKeep : EpiBase {
  static_assert(TL::MB % 4 == 0 && TL::NB % 4 == 0, "features and tokens are taken 64 at a time");
  EpiMoments<TL> mom;
  float* YT;
  int64_t ldt, tb, batch_stride;  // batch_stride in elements of YT
  __device__ __forceinline__ void operator()(floatx4 (&acc)[TL::MB][TL::NB], int batch, int tm,
                                             int tn, int ks, int m0, int n0) const {
    mom(acc, batch, tm, tn, ks, m0, n0);
    const Frag<TL> f;
#pragma unroll
    for (int g = 0; g < TL::NB / 4; ++g) {
      const int group0 = n0 + f.wn * TL::WTN + 64 * g;
      if (group0 >= ldt) return;
      const int64_t pos0 = group0 + (f.l16 << 2);
      const int64_t blk = pos0 / tb;
      float* out = YT + (int64_t)batch * batch_stride + blk * mom.d * tb + (pos0 - blk * tb);
#pragma unroll
      for (int mb = 0; mb < TL::MB; ++mb) {
        if (m0 + f.m_block(mb) < mom.d) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const floatx4 v = {acc[mb][4 * g][r], acc[mb][4 * g + 1][r], acc[mb][4 * g + 2][r], acc[mb][4 * g + 3][r]};
            *reinterpret_cast<floatx4*>(out + (int64_t)(m0 + f.m_of(mb, r)) * tb) = v;
          }
        }
      }
    }
  }
};

// ---- plain fp32 store, optionally into split-K partial slabs ---------------------
// C[ks*split_stride + batch*batch_stride + m*ldc + n]
template <class TL>
struct EpiStore : EpiBase {
  float* C;
  int64_t ldc, batch_stride, split_stride;
  int M, N;
  // operands swapped: a lane owns four consecutive columns of one row of every block, so the tile leaves as 16-byte
  // stores straight from the accumulators (a store instruction covers 16 rows x 64 bytes, the block beside it the
  // other half of those 128-byte lines)
  static constexpr bool kSwap = true;
  __device__ __forceinline__ void operator()(floatx4 (&acc)[TL::MB][TL::NB], int batch, int,
                                             int, int ks, int m0, int n0) const {
    const Frag<TL> f;
    float* base = C + (int64_t)ks * split_stride + (int64_t)batch * batch_stride;
    // 16-byte stores need aligned rows and whole groups of 4 columns inside N (uniform over the launch)
    const bool vec = ((reinterpret_cast<uintptr_t>(base) | (uintptr_t)(ldc * 4)) & 15) == 0 && (N & 3) == 0;
#pragma unroll
    for (int mb = 0; mb < TL::MB; ++mb) {
      const int m = m0 + f.m_row(mb);
      if (m < M) {
        float* row = base + (int64_t)m * ldc;
#pragma unroll
        for (int nb = 0; nb < TL::NB; ++nb) {
          const int n = n0 + f.n_quad(nb);
          const floatx4 v = acc[mb][nb];
          if (vec) {
            if (n < N) *reinterpret_cast<floatx4*>(row + n) = v;
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (n + r < N) row[n + r] = v[r];
          }
        }
      }
    }
  }
};

// Max of |x| taken on bit patterns: for non-negative floats the unsigned order is the
// numeric order, +inf sits above every finite value and NaN above +inf, so a NaN
// anywhere survives the reduction instead of being dropped as fmaxf would.
__device__ __forceinline__ unsigned abs_bits(float v) { return __float_as_uint(v) & 0x7fffffffu; }
__device__ __forceinline__ unsigned umax(unsigned a, unsigned b) { return a > b ? a : b; }
__device__ __forceinline__ unsigned wave_umax(unsigned v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = umax(v, (unsigned)__shfl_xor((int)v, o));
  return v;
}

// *word = max(*word, v over the four waves of the workgroup); the LDS of the main loop is free behind the first barrier.  One atomic a
// workgroup, and none where the word is already as large: all of them go to one address and take it about 10 ns each (256
// workgroups of a 512 x 512 product, one atomic a wave: 11 of 20 us).
__device__ __forceinline__ void workgroup_umax(unsigned v, unsigned* word) {
  extern __shared__ __align__(16) char lds[];
  unsigned* sh = reinterpret_cast<unsigned*>(lds);
  v = wave_umax(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    v = umax(umax(sh[0], sh[1]), umax(sh[2], sh[3]));
    if (v > __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(word, v);
  }
}

// ---- fp32 products of the retraction from fp16 heads and tails (split3_kernel) --------------------
// Words of one problem.  Every operand is multiplied by a power of two, chosen on the device from its largest magnitude; here are
// the exponents, so that a product comes back in one exact step (two factors 2^-k one after the other overflow with a gradient of 2^110, and a
// factor has to end at 2^-126 where a gradient of 2^-120 needs more).
struct SplitScales {
  int g, r;        // of the two operands of G R^T
  unsigned max_m;  // bit pattern of max |G R^T|
  int u, b;        // of U and B
};
// The k with 2^k |x| < 2^exponent for magnitudes up to that of `bits` (a non-negative float's bit pattern); 0 for zero, infinities and
// NaN, which come out as they are.
__device__ __forceinline__ int split_exponent(unsigned bits, int exponent) {
  const int e = (int)(bits >> 23);
  return bits == 0u || e >= 255 ? 0 : exponent - (e - 126);
}
// y = 2^k x -> fp16 head and tail, together within 2^-23 |y| of y while |y| >= 2^-2 and within 2^-25 below: 2^-40 of the operand's
// largest magnitude with exponent 15, 2^-32 (U) with 7.
__device__ __forceinline__ void split_f16(float x, int k, _Float16& hi, _Float16& lo) {
  const float y = ldexpf(x, k);
  hi = (_Float16)y;
  lo = (_Float16)(y - (float)hi);
}

// C = 2^shift * acc / (the two scales), and optionally the largest magnitude of it.  d x d, rows of d.
template <class TL>
struct EpiStoreScaled : EpiBase {
  float* C;
  const int *exp_a, *exp_b;  // of problem 0
  unsigned* max_word;        // of problem 0, or null
  int d, shift;
  static constexpr bool kSwap = true;
  __device__ __forceinline__ void operator()(floatx4 (&acc)[TL::MB][TL::NB], int batch, int, int, int, int m0, int n0) const {
    constexpr int kWords = sizeof(SplitScales) / 4;
    const Frag<TL> f;
    const int e = shift - exp_a[kWords * batch] - exp_b[kWords * batch];
    float* base = C + (int64_t)batch * d * d;
    unsigned most = 0u;
#pragma unroll
    for (int mb = 0; mb < TL::MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < TL::NB; ++nb) {
        const int m = m0 + f.m_row(mb), n = n0 + f.n_quad(nb);
        if (m < d && n < d) {
          floatx4 v;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            v[r] = ldexpf(acc[mb][nb][r], e);
            most = umax(most, abs_bits(v[r]));
          }
          *reinterpret_cast<floatx4*>(base + (int64_t)m * d + n) = v;
        }
      }
    if (max_word) workgroup_umax(most, max_word + kWords * batch);
  }
};

// ---- Cayley fixed point, in transposed space ---------------------------------------
// acc = U_k * B^T.  Zt_new = Rt - acc;  U_{k+1} = Rt + Zt_new;
// delta[it] = max |Zt_new - Zt_old| (bit pattern of a non-negative float, max is
// order independent so the result is deterministic).
// kHeadCut, the sign bit of a change: the fp16 head of the first iteration's D_1 was cut off (EpiCayleyIter, phase 0).  What is cut off is
// larger than what is not, so that it goes with the largest magnitude.
// When an iteration counts as converged.  The map is linear, Z_k+1 - Z_k = -B (Z_k - Z_k-1), so the
// changes shrink geometrically with the spectral radius rho of B = (lr/2) A and the iterate just written
// is within d_k rho / (1 - rho) of the fixed point (d_k = max |Z_k - Z_k-1|).  rho is estimated from the
// changes themselves.  Even and odd powers of a skew matrix have different patterns (for a low-rank
// gradient, B^2k is concentrated on a few entries and B^2k+1 is not, or the other way round), so that
// successive maxima alternate between two levels: the ratio over TWO steps, d_k / d_k-2 = rho^2, does not
// see that and is used as soon as three changes are there; with two, the one-step ratio.
//  - first iteration: converged only if the whole step is below the tolerance;
//  - 4 d_k rho / (1 - rho) <= tol (four times the distance bound), rho < 0.95; for rho < 0.2 this
//    accepts an iterate before its own change is below the tolerance and saves the product that would only
//    confirm it, for slow contractions it asks for more than d_k <= tol: what is left of the series then
//    still matters for max |R^T R - I|;
//  - the rounding floor: the change is small (within 64 tolerances) and has stopped shrinking over both of
//    the last two steps (for the three-term products the floor lies at a few 1e-7 and would never pass
//    a fixed fp32-sized tolerance).
// d1, d0, d00: changes of iterations k, k-1, k-2; nprev: how many of d0, d00 exist (0, 1 or 2).
constexpr unsigned kHeadCut = 0x80000000u;
__device__ __forceinline__ bool cayley_converged_hist(float d1, float d0, float d00, int nprev, float tol) {
  if (nprev == 0) return d1 <= tol;
  if (d1 == 0.f) return true;
  const float rho = nprev >= 2 ? sqrtf(d1 / d00) : d1 / d0;
  if (rho < 0.95f && 4.f * d1 * rho <= tol * (1.f - rho)) return true;
  if (nprev < 2 || !(d1 <= 64.f * tol)) return false;
  return d1 >= 0.9f * d0 && d1 >= 0.8f * d00;
}
// The changes of a problem as bits.  F16: the first may carry kHeadCut, and the second iteration ends a step only with a change of at most second_tol
// that follows from a whole head (EpiCayleyIter, phase 1).  fp32 has neither: the two tests cost its steps 0.4 %, in every launch.
template <bool F16>
__device__ __forceinline__ float cayley_change(unsigned bits) { return __uint_as_float(F16 ? bits & ~kHeadCut : bits); }
// (the changes are read past the caches of this XCD: inside cayley_iterate_kernel others have just written them; not asked for k < 2 with F16)
template <bool F16>
__device__ __forceinline__ bool cayley_converged_now(const unsigned* dl, int k, float tol) {
  auto at = [&](int i) { return cayley_change<F16>(__hip_atomic_load(dl + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)); };
  return cayley_converged_hist(at(k), k > 0 ? at(k - 1) : 0.f, k > 1 ? at(k - 2) : 0.f, k > 1 ? 2 : k, tol);
}
template <bool F16>
__device__ __forceinline__ bool cayley_converged(const unsigned* dl, int k, float tol, float second_tol) {
  auto at = [&](int i) { return cayley_change<F16>(dl[i]); };
  if (F16 && k == 1 && ((dl[0] & kHeadCut) != 0u || !(at(1) <= second_tol))) return false;
  return cayley_converged_hist(at(k), k > 0 ? at(k - 1) : 0.f, k > 1 ? at(k - 2) : 0.f, k > 1 ? 2 : k, tol);
}

// fp32: Zt and Unew as above.  As the epilogue of a launch of its own it returns at once when iteration
// it - 1 or an earlier one has converged.  (cayley_iterate_kernel sets `it` and the two targets.)
//
// fp16 heads and tails: Zt holds the displacement D = Z - Rt instead, which is what a step needs to be exact in (R + D is rounded once,
// by cayley_finish_kernel).  D_1 = - U_0 B^T, U_0 = 2 Rt, and from there D_k+1 = - U_k B^T, U_k = 2 Rt + D_k, in three terms; but the
// change of the second iteration is D_2 - D_1 = - D_1 B^T, and in one term, D_1 and B as heads alone (2^-12 of a value), it is as good
// as the first while it is small: an error of 2^-12 |D_2 - D_1|, random from entry to entry.  So phase 0 (the first iteration) leaves D and
// the head of D_1, phase 1 adds the change, and a second iteration counts as the last one only if its largest change is within 5e-4 of the
// root mean square of R's entries, 1/sqrt(d); from the third on (phase 2) U comes back, from cayley_u_kernel the first time, and what the
// second left out goes with it.  A dense B of norm rho changes the entries by 0.7 rho^2 of it then and stops 0.7 rho^3 short, 2^-12 / rho times
// what the heads leave out, and both are below the rounding of R at rho = 2e-3.  Error of R against 64 bits before / now over d = 1024 .. 4096, Haar,
// near-identity R and I, Gaussian, learned and log-normal gradients, (lr / 2) ||A|| = 5e-4 .. 0.3 (315 steps): 1.7e-8 .. 6.0e-7 in both, 0.999 to
// 1.003 times the former but for two steps of 11 iterations and more.
//   Usual steps end there (the change is 1e-11 to 1e-6): step in us, three terms in both / this: d = 1152, pooled loss and Adam, 10007 tokens 283 / 256,
//   2048, 65536 tokens 1134 / 1083, 4096, 131072 tokens 7392 / 7069.
template <class TL, int PHASE = 2>
struct EpiCayleyIter {
  static constexpr bool kF16 = sizeof(typename TL::T) == 2;
  const float* Rt;
  float* Zt;
  float* Unew;
  _Float16* Usplit;  // U as [head | tail] (phase 0: the head of D_1, rows of d)
  const SplitScales* scales = nullptr;
  unsigned* delta;  // [batch][max_iters]
  int d, it, max_iters;
  float tol, second_tol;
  const float* bscale = nullptr;  // acc is scaled by bscale[4 * batch + 3] when given (Cayley Adam)
  static constexpr bool kSwap = true;  // four consecutive columns of a row per lane: 16-byte accesses
  __device__ __forceinline__ bool skip(int batch) const {
    if (it == 0 || !cayley_converged<kF16>(delta + (int64_t)batch * max_iters, it - 1, tol, second_tol)) return false;
    // a zero change counts as converged: later launches return too
    if (blockIdx.x == 0 && threadIdx.x == 0) delta[(int64_t)batch * max_iters + it] = 0u;
    return true;
  }
  __device__ __forceinline__ void operator()(floatx4 (&acc)[TL::MB][TL::NB], int batch, int,
                                             int, int, int m0, int n0) const {
    apply<false>(acc, batch, m0, n0);
  }
  // The exponent of the head of D_1 = bs D', bs = f 2^eb: |D'| <= 2 sqrt(d) max |B|, the rows of R being of norm one, and 2^kb |B| < 2^15, so that
  // 2^(kb - half - 1) leaves it below 2^15, half = log2(d) / 2 rounded up.  Rows longer than two can be cut off at the largest fp16 value: the
  // change that follows from the head is too small then, and no second iteration counts as the last (kHeadCut; accepted by its own size, a step of
  // rows of norm 100 and a B of rank two along them ended 4e-6 of its norm off).
  static __device__ __forceinline__ int head_exponent(int kb, int eb, int d) { return kb - eb - (33 - __clz(d - 1)) / 2 - 1; }
  template <bool PAST_L2>
  __device__ __forceinline__ void apply(floatx4 (&acc)[TL::MB][TL::NB], int batch, int m0, int n0) const {
    typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
    const Frag<TL> f;
    const int64_t bo = (int64_t)batch * d * d;
    const float bs = bscale ? bscale[4 * batch + 3] : 1.f;
    int ku = 0, kb = 0, kd = 0, eb = 0;
    float bm = 1.f;
    if constexpr (kF16) {
      ku = scales[batch].u;
      kb = scales[batch].b;
      bm = frexpf(bs, &eb);
      kd = head_exponent(kb, eb, d);
    }
    unsigned dmax = 0u;
#pragma unroll
    for (int mb = 0; mb < TL::MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < TL::NB; ++nb) {
        const int m = m0 + f.m_row(mb), n = n0 + f.n_quad(nb);
        if (m < d && n < d) {  // d is a multiple of 128: all four columns are inside or none
          const int64_t idx = bo + (int64_t)m * d + n;
          floatx4 z;
          if constexpr (!kF16) {
            const floatx4 rt = *reinterpret_cast<const floatx4*>(Rt + idx);
            const floatx4 zo = *reinterpret_cast<const floatx4*>(Zt + idx);
            floatx4 u;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              z[r] = rt[r] - bs * acc[mb][nb][r];
              dmax = umax(dmax, abs_bits(z[r] - zo[r]));
              u[r] = rt[r] + z[r];
            }
            put<PAST_L2>(Zt + idx, z);
            put<PAST_L2>(Unew + idx, u);
          } else if constexpr (PHASE == 0) {
            f16x4 head;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              z[r] = -bs * ldexpf(acc[mb][nb][r], -(ku + kb));
              dmax = umax(dmax, abs_bits(z[r]));
              head[r] = (_Float16)__builtin_amdgcn_fmed3f(ldexpf(z[r], kd), -65504.f, 65504.f);
            }
            *reinterpret_cast<floatx4*>(Zt + idx) = z;
            *reinterpret_cast<f16x4*>(Usplit + idx) = head;
          } else if constexpr (PHASE == 1) {
            z = *reinterpret_cast<const floatx4*>(Zt + idx);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float change = -bm * ldexpf(acc[mb][nb][r], eb - (kd + kb));
              z[r] += change;
              dmax = umax(dmax, abs_bits(change));
            }
            *reinterpret_cast<floatx4*>(Zt + idx) = z;
          } else {
            const floatx4 rt = *reinterpret_cast<const floatx4*>(Rt + idx);
            const floatx4 zo = *reinterpret_cast<const floatx4*>(Zt + idx);
            f16x4 hi, lo;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              z[r] = -bs * ldexpf(acc[mb][nb][r], -(ku + kb));
              dmax = umax(dmax, abs_bits(z[r] - zo[r]));
              _Float16 h, l;
              split_f16(fmaf(2.f, rt[r], z[r]), ku, h, l);
              hi[r] = h;
              lo[r] = l;
            }
            put<PAST_L2>(Zt + idx, z);
            const int64_t so = 2 * bo + (int64_t)m * 2 * d + n;
            put<PAST_L2>(Usplit + so, hi);
            put<PAST_L2>(Usplit + so + d, lo);
          }
        }
      }
    if (kF16 && PHASE == 0 && !(ldexpf(__uint_as_float(dmax), kd) <= 65504.f)) dmax |= kHeadCut;
    workgroup_umax(dmax, &delta[(int64_t)batch * max_iters + it]);
  }
};

// ---- the later iterations in one launch ------------------------------------------------------
// Control words of one problem, all zero at the start: done[k] = tiles of iteration k that are complete, claim[t] = how many
// iterations of tile t have been taken.
constexpr int kCayleyControlWords = 64;  // done[0 .. 31], stop at 32; claim[] behind them

// Iterations k = it0, it0 + 1, ... of  Zt <- Rt - U_k B^T, U_k+1 = Rt + Zt  until they converge, with the dependency of each on
// all tiles of the one before inside the launch.  grid = (workgroups, problems); a workgroup owns the tiles w, w + gridDim.x, ...
//
// No workgroup relies on another one being resident: a tile of an iteration is taken by raising claim[t]; a workgroup takes
// its own ones as the iteration opens, and while it waits for the others it takes whatever nobody has taken.  So every tile
// that is waited for is in the hands of a running workgroup, whatever else runs on the chip.  (The wait ends after
// kCayleyWaitTicks all the same; the step then counts as not converged.)
//
// The results of a tile become visible with a release at device scope by one thread behind the workgroup's stores, or (PAST_L2) are
// stored past the L2: the stores of a wave are waited for, the barrier gathers the waves, and done[] is raised behind it.  They are
// acquired at device scope behind the wait; done[], claim[] and the changes are atomics.
//
// Why one launch: the host cannot know when the iteration has converged, so a launch per iteration means all 32 of them, and one
// that only finds the convergence flag set costs 2 to 3 us.  Why not for the first ones: a release and an acquire per tile write
// back and drop an XCD's L2 while other workgroups work from it (cayley_own_launches has the figures).  PAST_L2 leaves the acquire: better
// from 200 tiles of 64 x 64 on, 24 iterations, all but three inside, us, release / past the L2: d = 256, 16 problems (256 tiles) 429 / 361, 64 (1024) 1510 / 919,
// 512, 8 (512) 986 / 831, 896, 2 (392) 1369 / 1308, fp16 1024 (256) 912 / 863; but 256, 1 (16) 268 / 319, 512 (64) 408 / 467, 768 (144) 609 / 657, and
// 256 x 256 tiles, d = 4096, 9500 / 10500.
constexpr long long kCayleyWaitTicks = 20ll * 100000000;  // 20 s of the 100 MHz counter

template <class TL, bool PAST_L2>
__global__ __launch_bounds__(TL::NT) void cayley_iterate_kernel(GemmShape g, EpiCayleyIter<TL> epi, const typename TL::T* U0,
                                                                const typename TL::T* U1, unsigned* control, int64_t control_stride, int it0) {
  extern __shared__ __align__(16) char lds[];
  using T = typename TL::T;
  const int batch = blockIdx.y, tiles = g.tiles_total;
  unsigned* done = control + (int64_t)batch * control_stride;
  unsigned* stop = done + 32;
  unsigned* claim = done + kCayleyControlWords;
  unsigned* delta = epi.delta + (int64_t)batch * epi.max_iters;
  const T* B = static_cast<const T*>(g.B) + (int64_t)batch * g.batch_stride_b;
  int* said = reinterpret_cast<int*>(lds);  // {tile or -1, iteration}, from wave 0 (the LDS is free between two tiles)
  auto load = [](const unsigned* p) __attribute__((always_inline)) {
    return (unsigned)__builtin_amdgcn_readfirstlane((int)__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  };

  if (cayley_converged_now<EpiCayleyIter<TL>::kF16>(delta, it0 - 1, epi.tol)) return;
  int it = it0, own = blockIdx.x;  // wave 0: the open iteration, the next of this workgroup's tiles in it
  bool looked = false;           // ... has just found a tile of somebody else's: look for the next one at once
  // tile t of iteration `it`, if nobody has it (wave 0)
  auto take = [&](int t) __attribute__((always_inline)) {
    int got = 0;
    if (threadIdx.x == 0) got = atomicCAS(claim + t, (unsigned)(it - it0), (unsigned)(it - it0) + 1) == (unsigned)(it - it0);
    return __builtin_amdgcn_readfirstlane(got) != 0;
  };
  // the next tile for this workgroup, -1 when there is none left (wave 0)
  auto next_tile = [&]() __attribute__((always_inline)) {
    for (;;) {
      while (own < tiles) {
        const int t = own;
        own += gridDim.x;
        if (take(t)) return t;
      }
      const long long t0 = __builtin_amdgcn_s_memrealtime();
      for (int polls = looked ? 15 : 0; load(done + it) < (unsigned)tiles; ++polls) {
        if ((polls & 15) == 15) {
          if (load(stop) != 0u) return -1;
          if ((long long)__builtin_amdgcn_s_memrealtime() - t0 > kCayleyWaitTicks) {
            if (threadIdx.x == 0) {
              __hip_atomic_store(stop, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              for (int k = it; k < epi.max_iters; ++k) atomicMax(delta + k, 0x7fc00000u);
            }
            return -1;
          }
          int mine = -1;
          for (int t = threadIdx.x; t < tiles; t += 64)
            if (mine < 0 && __hip_atomic_load(claim + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)(it - it0)) mine = t;
          const unsigned long long found = __ballot(mine >= 0);
          if (found) {
            const int t = __builtin_amdgcn_readlane(mine, __builtin_ctzll(found));
            looked = true;
            if (take(t)) return t;
          }
        }
        __builtin_amdgcn_s_sleep(2);
      }
      looked = false;
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      if (it + 1 == epi.max_iters || cayley_converged_now<EpiCayleyIter<TL>::kF16>(delta, it, epi.tol)) return -1;
      ++it;
      own = blockIdx.x;
    }
  };

#pragma unroll 1
  for (;;) {
    __syncthreads();
    if (threadIdx.x < 64) {
      const int t = next_tile();
      if (threadIdx.x == 0) {
        said[0] = t;
        said[1] = it;
      }
    }
    __syncthreads();
    const int t = __builtin_amdgcn_readfirstlane(said[0]), k = __builtin_amdgcn_readfirstlane(said[1]);
    __syncthreads();
    if (t < 0) return;
    int tm, tn;
    tile_in_bands(g, (tiles & 7) ? t : (t & 7) * (tiles >> 3) + (t >> 3), tm, tn);  // (neighbours on one XCD, as in tile_of_block)
    const int m0 = tm * TL::BM, n0 = tn * TL::BN;
    floatx4 acc[TL::MB][TL::NB];
#pragma unroll
    for (int mb = 0; mb < TL::MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < TL::NB; ++nb) acc[mb][nb] = floatx4{0.f, 0.f, 0.f, 0.f};
    settle_all<TL>(acc);
    gemm_mainloop<TL, false, false, true>((k & 1 ? U1 : U0) + (int64_t)batch * g.batch_stride_a, g.lda, g.M, m0, B, g.ldb, g.N, n0, 0,
                                          g.slabs_total, g.slabs_per_block, 0, acc, lds, 0, 0);
    settle_all<TL>(acc);
    EpiCayleyIter<TL> e = epi;
    e.it = k;
    T* next = const_cast<T*>(k & 1 ? U0 : U1);
    if constexpr (sizeof(T) == 2) e.Usplit = next;
    else e.Unew = next;
    e.template apply<PAST_L2>(acc, batch, m0, n0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's stores (and its change) have reached the L2, or the memory behind it
    __syncthreads();
    if (threadIdx.x == 0) {
      if constexpr (!PAST_L2) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      __hip_atomic_fetch_add(done + k, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// ---- orthogonality check: max |acc_mn| over m != n -----------------------------------
// The diagonal (sums of squares close to 1, where fp32 accumulation loses ~1e-7 per
// entry) is left to ortho_diag_kernel, which sums in fp64.
template <class TL>
struct EpiOrtho : EpiBase {
  unsigned* err;  // [batch], bit pattern of a non-negative float, zeroed before launch
  int d;
  __device__ __forceinline__ void operator()(floatx4 (&acc)[TL::MB][TL::NB], int batch, int,
                                             int, int, int m0, int n0) const {
    const Frag<TL> f;
    unsigned e = 0u;
#pragma unroll
    for (int mb = 0; mb < TL::MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < TL::NB; ++nb) {
        const int n = n0 + f.n_of(nb);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = m0 + f.m_of(mb, r);
          if (m < d && n < d && m != n) e = umax(e, abs_bits(acc[mb][nb][r]));
        }
      }
    workgroup_umax(e, &err[batch]);
  }
};

// ---- fake-quant pass A: per-token max |y| -----------------------------------------
// same orientation as EpiMoments; part[(batch*P + p)*n_tokens + token]
template <class TL, bool PAST_L2 = false>
struct EpiAmax : EpiBase {
  static_assert(TL::MB % 4 == 0 && TL::NB % 4 == 0, "features and tokens are taken 64 at a time");
  float* part;
  int n_tokens, d, P;
  __device__ __forceinline__ void operator()(floatx4 (&acc)[TL::MB][TL::NB], int batch, int tm,
                                             int, int, int m0, int n0) const {
    const Frag<TL> f(thread_id<PAST_L2>());
    const int p = tm * TL::WGM + f.wm;
#pragma unroll
    for (int g = 0; g < TL::NB / 4; ++g) {  // 64 tokens: lane l ends up with token l of them
      float a[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        a[k] = 0.f;
#pragma unroll
        for (int mb = 0; mb < TL::MB; ++mb)
          if (m0 + f.m_block(mb) < d) {
#pragma unroll
            for (int r = 0; r < 4; ++r) a[k] = fmaxf(a[k], fabsf(acc[mb][4 * g + k][r]));
          }
      }
      const float v = quarter_reduce4<OpMax>(a[0], a[1], a[2], a[3]);
      const int token = n0 + f.wn * TL::WTN + 64 * g + f.lane;
      if (token < n_tokens && p < P) {
        if constexpr (PAST_L2) __hip_atomic_store(&part[((int64_t)batch * P + p) * n_tokens + token], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else part[((int64_t)batch * P + p) * n_tokens + token] = v;
      }
    }
  }
};

// ---- fake-quant pass B: quantise the recomputed y ----------------------------------
// Same orientation as the moment epilogue (token on the lane, features on the registers): the
// scale and its reciprocal are taken once per token, the error sums accumulate in registers and
// meet only the other lane quarters, and the codes leave as 16-byte stores (the four lanes of a
// token exchange packed words over four blocks first).  q = clamp(rint(y * (1/s)), -7, 7) in fp32;
// pe[(batch*P + p)*n_tokens + token] = {sum (y - q s)^2, sum y^2} over the wave's feature rows.
template <class TL, bool PAST_L2 = false>
struct EpiQuant : EpiBase {
  static_assert(TL::MB % 4 == 0 && TL::NB % 4 == 0, "features and tokens are taken 64 at a time");
  const float* scales;  // [batch][n_tokens]
  int8_t* codes;        // [batch][n_tokens][d] or null
  float2* err_part;     // or null
  int n_tokens, d, P;
  __device__ __forceinline__ void operator()(floatx4 (&acc)[TL::MB][TL::NB], int batch, int tm,
                                             int, int, int m0, int n0) const {
    apply(acc, batch, tm, m0, n0, [&](int t) __attribute__((always_inline)) {
      const float s = n0 + t < n_tokens ? scales[(int64_t)batch * n_tokens + n0 + t] : 0.f;
      return make_float2(s, s > 0.f ? __fdiv_rn(1.0f, s) : 0.f);
    });
  }
  // scale_of(t): the scale of token n0 + t and its reciprocal (0 where the scale is not positive)
  template <class ScaleOf>
  __device__ __forceinline__ void apply(floatx4 (&acc)[TL::MB][TL::NB], int batch, int tm, int m0, int n0, ScaleOf scale_of) const {
    const Frag<TL> f(thread_id<PAST_L2>());
    const int p = tm * TL::WGM + f.wm;
#pragma unroll
    for (int g = 0; g < TL::NB / 4; ++g) {
      float e2[4], y2[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int token = n0 + f.n_of(4 * g + k);
        const bool tv = token < n_tokens;
        const float2 scale = scale_of(token - n0);
        const float s = scale.x, rinv = scale.y;
        const float top = s > 0.f ? 7.f : 0.f;  // a row with scale 0 gets codes 0
        int8_t* crow = codes + ((int64_t)batch * n_tokens + token) * d;
        e2[k] = 0.f; y2[k] = 0.f;
#pragma unroll
        for (int m4 = 0; m4 < TL::MB / 4; ++m4) {
          if (m0 + f.m_block(4 * m4) < d) {  // d is a multiple of 128: the four blocks are inside together
            float pk[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              unsigned t[4];
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                // clamp(rint(v)) = rint(clamp(v)) for whole bounds; 1.5 2^23 + v has rint(v) (ties to even) in its low bits
                const float y = acc[4 * m4 + i][4 * g + k][e];
                const float v = __builtin_amdgcn_fmed3f(__fmul_rn(y, rinv), -top, top);
                const float m = __fadd_rn(v, 12582912.f);
                t[e] = __float_as_uint(m);
                const float diff = fmaf(-__fsub_rn(m, 12582912.f), s, y);
                e2[k] = fmaf(diff, diff, e2[k]);
                y2[k] = fmaf(y, y, y2[k]);
              }
              const unsigned lo = __builtin_amdgcn_perm(t[1], t[0], 0x0c0c0400u), hi = __builtin_amdgcn_perm(t[3], t[2], 0x04000c0cu);
              pk[i] = __uint_as_float(lo | hi);
            }
            // word i of quarter c = features 16 i + 4 c .. + 3 of these 64: transposed among the four lanes of the
            // token, quarter c holds all 16 bytes of block c
            swap_halves(pk[0], pk[2]);
            swap_halves(pk[1], pk[3]);
            swap_quarters(pk[0], pk[1]);
            swap_quarters(pk[2], pk[3]);
            const uintx4 out = {__float_as_uint(pk[0]), __float_as_uint(pk[1]), __float_as_uint(pk[2]), __float_as_uint(pk[3])};
            if (codes && tv) *reinterpret_cast<uintx4*>(crow + m0 + f.m_block(4 * m4) + 16 * f.q) = out;
          }
        }
      }
      if (err_part) {
        const float2 v = make_float2(quarter_reduce4<OpAdd>(e2[0], e2[1], e2[2], e2[3]),
                                     quarter_reduce4<OpAdd>(y2[0], y2[1], y2[2], y2[3]));
        const int token = n0 + f.wn * TL::WTN + 64 * g + f.lane;
        if (token < n_tokens && p < P) {
          if constexpr (PAST_L2)
            __hip_atomic_store(reinterpret_cast<uint64_t*>(&err_part[((int64_t)batch * P + p) * n_tokens + token]), __builtin_bit_cast(uint64_t, v),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          else
            err_part[((int64_t)batch * P + p) * n_tokens + token] = v;
        }
      }
    }
  }
};

}  // namespace kt
