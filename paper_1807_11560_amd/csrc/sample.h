// Periodic sampling of a grid field, shared by the transport kernels.
#pragma once

#include "common.h"

namespace lddmm {

// a mod N in [0, N); points rarely leave the grid, so the division is rare
__device__ __forceinline__ int wrap(int a, int N) {
  if ((unsigned)a >= (unsigned)N) {
    a %= N;
    if (a < 0) a += N;
  }
  return a;
}

// The cell of voxel coordinates X (floor, periodic): the offsets of its four
// rows, (a0, a1), (a0, b1), (b0, a1), (b0, b1) with b = a + 1, its first column
// a2, the floors as they are, and the fractional parts.  (Products of 24 bits: N0, N1 <= 2048, N2 <= 256.)
struct Cell {
  unsigned r[4];
  int a2;
  int f0, f1, f2;
  float w0, w1, w2;
};
template <class G>
__device__ __forceinline__ Cell cell_at(float X0, float X1, float X2, int i0, int i1, int i2, G gs) {
  const int N0 = gs.N0(), N1 = gs.N1(), N2 = gs.N2();
  // a non-finite coordinate must not turn into an out-of-range index
  if (!isfinite(X0)) X0 = (float)i0;
  if (!isfinite(X1)) X1 = (float)i1;
  if (!isfinite(X2)) X2 = (float)i2;
  const float f0 = floorf(X0), f1 = floorf(X1), f2 = floorf(X2);
  const int a0 = wrap((int)f0, N0), a1 = wrap((int)f1, N1);
  const int b0 = (a0 + 1 == N0) ? 0 : a0 + 1;
  const int b1 = (a1 + 1 == N1) ? 0 : a1 + 1;
  Cell c;
  const unsigned p0 = __umul24(a0, N1), p1 = __umul24(b0, N1);
  c.r[0] = __umul24(p0 + a1, N2);
  c.r[1] = __umul24(p0 + b1, N2);
  c.r[2] = __umul24(p1 + a1, N2);
  c.r[3] = __umul24(p1 + b1, N2);
  c.a2 = wrap((int)f2, N2);
  c.f0 = (int)f0;
  c.f1 = (int)f1;
  c.f2 = (int)f2;
  c.w0 = X0 - f0;
  c.w1 = X1 - f1;
  c.w2 = X2 - f2;
  return c;
}

// The eight corners of a cell, v[2 q] and v[2 q + 1] those of row q: one 8-byte
// load per row (a cell that wraps around the last axis reads its far corner
// apart).
typedef float f2_u4 __attribute__((ext_vector_type(2), aligned(4)));
template <class G>
__device__ __forceinline__ void corners(const float* __restrict__ f, const Cell& c, float (&v)[8], G gs) {
  const int N2 = gs.N2();
  const bool edge = c.a2 == N2 - 1;
  const unsigned at = edge ? c.a2 - 1 : c.a2;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const f2_u4 t = *reinterpret_cast<const f2_u4*>(f + (size_t)(c.r[q] + at));
    v[2 * q] = edge ? t.y : t.x;
    v[2 * q + 1] = t.y;
  }
  if (edge) {
#pragma unroll
    for (int q = 0; q < 4; ++q) v[2 * q + 1] = f[c.r[q]];
  }
}

// Trilinear interpolation from the corners of a cell.
__device__ __forceinline__ float lerp8(const float (&v)[8], const Cell& c) {
  const float c00 = v[0] + c.w2 * (v[1] - v[0]);
  const float c01 = v[2] + c.w2 * (v[3] - v[2]);
  const float c10 = v[4] + c.w2 * (v[5] - v[4]);
  const float c11 = v[6] + c.w2 * (v[7] - v[6]);
  const float c0 = c00 + c.w1 * (c01 - c00);
  const float c1 = c10 + c.w1 * (c11 - c10);
  return c0 + c.w0 * (c1 - c0);
}

// The interpolant's slopes in the cell, per voxel of each axis.
__device__ __forceinline__ void slopes8(const float (&v)[8], const Cell& c, float* d0, float* d1, float* d2) {
  const float c00 = v[0] + c.w2 * (v[1] - v[0]), c01 = v[2] + c.w2 * (v[3] - v[2]);
  const float c10 = v[4] + c.w2 * (v[5] - v[4]), c11 = v[6] + c.w2 * (v[7] - v[6]);
  const float c0 = c00 + c.w1 * (c01 - c00), c1 = c10 + c.w1 * (c11 - c10);
  *d0 = c1 - c0;
  *d1 = (c01 - c00) + c.w0 * ((c11 - c10) - (c01 - c00));
  const float e00 = v[1] - v[0], e01 = v[3] - v[2], e10 = v[5] - v[4], e11 = v[7] - v[6];
  const float e0 = e00 + c.w1 * (e01 - e00), e1 = e10 + c.w1 * (e11 - e10);
  *d2 = e0 + c.w0 * (e1 - e0);
}

// Periodic trilinear interpolation of f at voxel coordinates X of the point
// (i0, i1, i2).
template <class G>
__device__ __forceinline__ float trilinear(const float* __restrict__ f, float X0, float X1, float X2, int i0,
                                           int i1, int i2, G gs) {
  const Cell c = cell_at(X0, X1, X2, i0, i1, i2, gs);
  float v[8];
  corners(f, c, v, gs);
  return lerp8(v, c);
}

// Point of thread (blockIdx.x blockDim.x + threadIdx.x) of plane blockIdx.y:
// false past the plane's end.
template <class G>
__device__ __forceinline__ bool plane_point(G gs, int* i0, int* i1, int* i2, long long* gi) {
  const unsigned p = blockIdx.x * blockDim.x + threadIdx.x, n = gs.N1() * gs.N2();
  *i0 = blockIdx.y;
  *i1 = p / (unsigned)gs.N2();
  *i2 = p - *i1 * gs.N2();
  *gi = (long long)blockIdx.y * n + p;
  return p < n;
}

}  // namespace lddmm
