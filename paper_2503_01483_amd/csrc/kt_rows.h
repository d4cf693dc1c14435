// kt_rows.h -- kurtosis loss and dL/dY of token-major fp32 rows (the fp32 path): Y [problem][ldt][d] as the forward product left
// it, G = dL/dY over it in place.
//
// One wave per row (d = 128: half a wave), the row in registers (16-byte loads, all in flight), statistics and gradient in one pass: bound by HBM,
// 8 bytes per value, by the latency of one row in small calls, or by the fp64 arithmetic of a row's statistics in many short rows.  The fp32 products take either operand with K as its row
// index, so neither Y, G nor X is ever transposed.  fp32 steps, us, with row sums in the forward epilogue (128 x 128 tiles), transposed
// copies of R, X and Y and three to five kernels between the products / this form: d = 256, 2048 tokens 93 / 59; 640, 1000 154 / 104;
// 512, 4096, pooled 171 / 137; 1024, 16384 723 / 663.
#pragma once
#include "kt_aux.h"

namespace kt {

// Sum over LANES neighbouring lanes, in each of them, in a fixed order.
template <int LANES>
__device__ __forceinline__ double lanes_sum(double v) {
#pragma unroll
  for (int o = LANES / 2; o >= 1; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// Calls f(chunk, value) for the float4s of a row this lane holds: v[CH] (d <= 4 LANES CH), or read again (CH = 0).
template <int CH, int LANES, class F>
__device__ __forceinline__ void for_row(const float4 (&v)[CH ? CH : 1], const float4* y4, int d, F f) {
  const int lane4 = 4 * (threadIdx.x & (LANES - 1));
  if constexpr (CH > 0) {
#pragma unroll
    for (int c = 0; c < CH; ++c)
      if (4 * LANES * c + lane4 < d) f(c, v[c]);
  } else {
    for (int c = 0; 4 * LANES * c + lane4 < d; ++c) f(c, y4[LANES * c]);
  }
}

// Rows of problem blockIdx.y, a workgroup 256 / LANES at a time.  Row loss (pool_part null): kappa, loss term and G over Y (want_grad).
// Pooled loss: part[row] = {mean, sums of c^2, c^3, c^4 about it} and the workgroup's sums of z^k, k = 1 .. 4 (pooled_row_sums).
// sum_part: [problem][gridDim.x] sums of the loss terms, or x 4 of z^k.  Rows n .. ldt - 1, the padding of the gradient product, are
// cleared.
template <int CH, int LANES>
__global__ __launch_bounds__(256) void loss_rows_kernel(float* __restrict__ Y, int ldt, int n, int d, float kappa_target,
                                                        float* __restrict__ row_kurt, double* __restrict__ sum_part, int want_grad,
                                                        float rms_eps, floatx4* __restrict__ part) {
  constexpr int ROWS = 256 / LANES;
  __shared__ double sh[ROWS][4];
  const int lane = threadIdx.x & (LANES - 1), group = threadIdx.x / LANES, batch = blockIdx.y;
  double sums[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
  for (int row = blockIdx.x * ROWS + group; row < ldt; row += ROWS * gridDim.x) {
    float4* y4 = reinterpret_cast<float4*>(Y + ((int64_t)batch * ldt + row) * d) + lane;
    if (row >= n) {
      if (want_grad)
        for (int c = 0; 4 * (LANES * c + lane) < d; ++c) y4[LANES * c] = make_float4(0.f, 0.f, 0.f, 0.f);
      continue;
    }
    float4 v[CH ? CH : 1];
#pragma unroll
    for (int c = 0; c < CH; ++c)
      if (4 * (LANES * c + lane) < d) v[c] = y4[LANES * c];
    double s = 0.0;
    for_row<CH, LANES>(v, y4, d, [&](int, const float4& t) { s += (double)((t.x + t.y) + (t.z + t.w)); });
    const double inv_d = 1.0 / (double)d;
    const float about = (float)(lanes_sum<LANES>(s) * inv_d);
    // sums about the mean rounded to fp32, four values at a time in fp32; the rest of the mean is shifted out in fp64
    double S1 = 0.0, S2 = 0.0, S3 = 0.0, S4 = 0.0;
    for_row<CH, LANES>(v, y4, d, [&](int, const float4& t) {
      const float e4[4] = {t.x, t.y, t.z, t.w};
      float s1 = 0.f, s2 = 0.f, s3 = 0.f, s4 = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float c = e4[e] - about, c2 = c * c;
        s1 += c;
        s2 += c2;
        s3 = fmaf(c2, c, s3);
        s4 = fmaf(c2, c2, s4);
      }
      S1 += (double)s1; S2 += (double)s2; S3 += (double)s3; S4 += (double)s4;
    });
    S1 = lanes_sum<LANES>(S1); S2 = lanes_sum<LANES>(S2); S3 = lanes_sum<LANES>(S3); S4 = lanes_sum<LANES>(S4);
    const double e = S1 * inv_d, dd = (double)d, mu = (double)about + e;
    const double M[3] = {S2 - dd * e * e, S3 - 3.0 * e * S2 + 2.0 * dd * e * e * e,
                         S4 - 4.0 * e * S3 + 6.0 * e * e * S2 - 3.0 * dd * e * e * e * e};
    if (part) {
      const floatx4 p = {(float)mu, (float)M[0], (float)M[1], (float)M[2]};
      double Z[4], inv_rho;
      pooled_row_sums(mu, M, d, (double)rms_eps, inv_rho, Z);
      if (lane == 0) part[(int64_t)batch * n + row] = p;
#pragma unroll
      for (int k = 0; k < 4; ++k) sums[k] += Z[k];
    } else {
      double kappa;
      const floatx4 c = row_coefficients(mu, M, n, d, kappa_target, kappa, sums[0]);
      if (row_kurt && lane == 0) row_kurt[(int64_t)batch * n + row] = (float)kappa;
      if (want_grad)
        for_row<CH, LANES>(v, y4, d, [&](int i, const float4& t) {
          y4[LANES * i] = make_float4(grad_value(t.x, c[0], c[1], c[2], c[3]), grad_value(t.y, c[0], c[1], c[2], c[3]),
                                   grad_value(t.z, c[0], c[1], c[2], c[3]), grad_value(t.w, c[0], c[1], c[2], c[3]));
        });
    }
  }
  const int words = part ? 4 : 1;
  if (lane == 0)
    for (int k = 0; k < words; ++k) sh[group][k] = sums[k];
  __syncthreads();
  if ((int)threadIdx.x < words) {
    double t = sh[0][threadIdx.x];
#pragma unroll
    for (int i = 1; i < ROWS; ++i) t += sh[i][threadIdx.x];
    sum_part[((int64_t)batch * gridDim.x + blockIdx.x) * words + threadIdx.x] = t;
  }
}

// Pooled loss: G over Y, from the row sums and the pooled statistics.  grid = (ceil(n LANES / 256), problems)
template <int LANES>
__global__ __launch_bounds__(256) void pooled_grad_rows_kernel(float* __restrict__ Y, int ldt, int n, int d, float rms_eps,
                                                               const floatx4* __restrict__ part, const double* __restrict__ gstat) {
  const int lane = threadIdx.x & (LANES - 1), row = blockIdx.x * (256 / LANES) + threadIdx.x / LANES, batch = blockIdx.y;
  if (row >= n) return;
  float4* y4 = reinterpret_cast<float4*>(Y + ((int64_t)batch * ldt + row) * d) + lane;
  const floatx4 p = part[(int64_t)batch * n + row];
  const double M[3] = {(double)p[1], (double)p[2], (double)p[3]};
  const floatx4 c = pooled_coefficients((double)p[0], M, d, rms_eps, gstat + 4 * batch);
#pragma unroll 4
  for (int i = 0; 4 * (LANES * i + lane) < d; ++i) {
    const float4 t = y4[LANES * i];
    y4[LANES * i] = make_float4(grad_value(t.x, c[0], c[1], c[2], c[3]), grad_value(t.y, c[0], c[1], c[2], c[3]),
                             grad_value(t.z, c[0], c[1], c[2], c[3]), grad_value(t.w, c[0], c[1], c[2], c[3]));
  }
}

}  // namespace kt
