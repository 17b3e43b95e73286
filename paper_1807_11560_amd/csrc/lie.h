// Pointwise products of the band Lie algebra on the padded grid.
#pragma once

#include "common.h"

namespace lddmm {

// --------------------------------------------- band Lie algebra products
// Group layout: 12 scalar fields of one vector field f: f_c at index c,
// d_i f_c at index 3 + 3c + i.
// (ad*_a mu)_i = sum_j (d_i a_j) mu_j + (d_j mu_i) a_j + mu_i (d_j a_j)
__device__ __forceinline__ void adstar_acc(float* o, const float* a, const float* mu, float s) {
  const float diva = a[3] + a[7] + a[11];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    float r = mu[i] * diva;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      r = fmaf(a[3 + 3 * j + i], mu[j], r);
      r = fmaf(mu[3 + 3 * i + j], a[j], r);
    }
    o[i] = fmaf(s, r, o[i]);
  }
}

// (ad_a b)_i = sum_j (d_j a_i) b_j - (d_j b_i) a_j
__device__ __forceinline__ void ad_acc(float* o, const float* a, const float* b, float s) {
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    float r = 0.f;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      r = fmaf(a[3 + 3 * i + j], b[j], r);
      r = fmaf(-b[3 + 3 * i + j], a[j], r);
    }
    o[i] = fmaf(s, r, o[i]);
  }
}

// (D~a * b)_i += sum_j (d_j a_i) b_j; ja[3 i + j] = d_j a_i
__device__ __forceinline__ void jac_acc(float* o, const float* ja, const float* b) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) o[i] = fmaf(ja[3 * i + j], b[j], o[i]);
}

// ((D~a)^T * r)_j += sum_i (d_j a_i) r_i
__device__ __forceinline__ void jact_acc(float* o, const float* ja, const float* r) {
#pragma unroll
  for (int j = 0; j < 3; ++j)
#pragma unroll
    for (int i = 0; i < 3; ++i) o[j] = fmaf(ja[3 * i + j], r[i], o[j]);
}

}  // namespace lddmm
