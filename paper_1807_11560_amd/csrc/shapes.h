// Problem sizes as seen by kernels, and the band symbols.
#pragma once

#include <math.h>

#include "common.h"

namespace lddmm {

// ---------------------------------------------------------------- shapes
// Sizes seen by a kernel: compile-time for the shapes this library is tuned
// for (index arithmetic then folds into constants), runtime otherwise.
struct BandDyn {
  static constexpr bool kStatic = false;
  int k0, k1, kh, m0, m1, m2;
  __device__ __forceinline__ int K0() const { return k0; }
  __device__ __forceinline__ int K1() const { return k1; }
  __device__ __forceinline__ int Kh() const { return kh; }
  __device__ __forceinline__ int M0() const { return m0; }
  __device__ __forceinline__ int M1() const { return m1; }
  __device__ __forceinline__ int M2() const { return m2; }
};
template <int K, int M>
struct BandIso {
  static constexpr bool kStatic = true;
  __device__ static constexpr int K0() { return K; }
  __device__ static constexpr int K1() { return K; }
  __device__ static constexpr int Kh() { return K / 2; }
  __device__ static constexpr int M0() { return M; }
  __device__ static constexpr int M1() { return M; }
  __device__ static constexpr int M2() { return M; }
};
struct GridDyn {
  static constexpr bool kStatic = false;
  int n0, n1, n2, k1, kh;
  __device__ __forceinline__ int N0() const { return n0; }
  __device__ __forceinline__ int N1() const { return n1; }
  __device__ __forceinline__ int N2() const { return n2; }
  __device__ __forceinline__ int K1() const { return k1; }
  __device__ __forceinline__ int Kh() const { return kh; }
};
template <int A, int B, int C, int K>
struct GridShape {
  static constexpr bool kStatic = true;
  __device__ static constexpr int N0() { return A; }
  __device__ static constexpr int N1() { return B; }
  __device__ static constexpr int N2() { return C; }
  __device__ static constexpr int K1() { return K; }
  __device__ static constexpr int Kh() { return K / 2; }
};
template <int N, int K>
using GridIso = GridShape<N, N, N, K>;

// L~ and K~ = 1 / L~ at the band slot (q0, q1, k2) (FP64, rounded once);
// kernels that need a few symbols per thread form them here instead of
// loading them from the tables.
__device__ __forceinline__ float2 band_symbols(int q0, int q1, int k2, int K0, int K1, int s, double alpha) {
  const int k0 = q0 < K0 / 2 ? q0 : q0 - K0;
  const int k1 = q1 < K1 / 2 ? q1 : q1 - K1;
  const double tp = 2.0 * M_PI;
  const double lap = tp * tp * ((double)k0 * k0 + (double)k1 * k1 + (double)k2 * k2);
  const double base = 1.0 + alpha * lap;
  double L = 1.0;
  for (int e = 0; e < s; ++e) L *= base;
  return make_float2((float)L, (float)(1.0 / L));
}

// ---------------------------------------------------------------- dispatch
inline bool band_iso(const Dims& d, int K, int M) {
  return d.K[0] == K && d.K[1] == K && d.K[2] == K && d.M[0] == M && d.M[1] == M && d.M[2] == M;
}
// Whether the band kernels of these sizes are instantiated (else: chain.hip).
inline bool band_instantiated(const Dims& d) {
  return band_iso(d, 32, 48) || band_iso(d, 16, 24) || band_iso(d, 24, 36);
}
inline bool grid_iso(const Dims& d, int N, int K) {
  return d.N[0] == N && d.N[1] == N && d.N[2] == N && d.K[1] == K && d.K[2] == K;
}
inline bool grid_is(const Dims& d, int A, int B, int C, int K) {
  return d.N[0] == A && d.N[1] == B && d.N[2] == C && d.K[1] == K && d.K[2] == K;
}
template <class F>
hipError_t with_grid(const Dims& d, F&& f) {
  // the measured volume, the 64^3 problem and the grids of the atlas
  // batch and of the differentiation volume, with bands 24^3 and 32^3
  if (grid_iso(d, 128, 32)) return f(GridIso<128, 32>{});
  if (grid_iso(d, 64, 16)) return f(GridIso<64, 16>{});
  if (grid_iso(d, 128, 24)) return f(GridIso<128, 24>{});
  if (grid_iso(d, 96, 24)) return f(GridIso<96, 24>{});
  if (grid_iso(d, 96, 32)) return f(GridIso<96, 32>{});
  if (grid_is(d, 144, 176, 144, 24)) return f(GridShape<144, 176, 144, 24>{});
  if (grid_is(d, 144, 176, 144, 32)) return f(GridShape<144, 176, 144, 32>{});
  if (grid_is(d, 160, 192, 160, 24)) return f(GridShape<160, 192, 160, 24>{});
  if (grid_is(d, 160, 192, 160, 32)) return f(GridShape<160, 192, 160, 32>{});
  return f(GridDyn{d.N[0], d.N[1], d.N[2], d.K[1], d.Kh});
}
inline bool grid_instantiated(const Dims& d) {
  bool is = false;
  (void)with_grid(d, [&](auto gs) {
    is = decltype(gs)::kStatic;
    return hipSuccess;
  });
  return is;
}
}  // namespace lddmm
