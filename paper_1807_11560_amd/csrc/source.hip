// The image-term sources and the image grid's forward transform.
#include "launch.h"
#include "mfma.h"
#include "sample.h"
#include "shapes.h"

namespace lddmm {
namespace {

// --------------------------------------------- forward stage 2 of a tile
// A tile of 16 rows of x1 of three real fields in LDS, vals[(3 fields) 16 rows
// of LV floats], the columns x2 = N2 .. 4 ceil(N2 / 4) - 1 zero: a wave takes
// (field, real or imaginary part, 16 kh) products D[row][kh] = sum_x2
// vals[row][x2] w(kh, x2), each a chain of matrix products and so the sequential
// sum over x2 (v_mfma_f32_16x16x4f32 adds its four products in turn), as scalar
// code forms it.  LV is an odd multiple of 4 floats: the 16 rows and 4 columns
// that a wave reads at once lie in different banks.  The table goes through
// LDS: a wave's operand of it from memory touches 16 rows per 16 lanes, 64
// cycles of the address unit.  The source kernel at 144x176x144 / band 24: 61 us
// with a thread per (row, kh), 44 with the table from memory, 30 so; at
// 180x210x180 / band 32 102, 51 and 56 (whose product phases overlap less).
__host__ __device__ constexpr int tile_ld(int N2) {
  const int q = (N2 + 3) / 4;
  return 4 * (q | 1);
}
constexpr int kSrcThreads = 512;
// The stage-2 table w(kh, x2) to LDS, ws[Kh][row_ld(N2)]: read along its rows.
__device__ __forceinline__ void stage_fwd2(float2* ws, const float2* __restrict__ w, int N2, int Kh) {
  const int n = Kh * N2, LW = row_ld(N2);
  constexpr int U = 4;
  for (int i0 = threadIdx.x; i0 < n; i0 += U * kSrcThreads) {
    float2 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = w[min(i0 + u * kSrcThreads, n - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * kSrcThreads;
      if (i < n) ws[(i / N2) * LW + i % N2] = v[u];
    }
  }
}
template <class Store>
__device__ __forceinline__ void fwd2_tile(const float* vals, const float2* ws, int N2, int Kh, int waves, Store store) {
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int LV = tile_ld(N2), kt = (Kh + 15) / 16, nk = (N2 + 3) / 4;
  for (int job = wave_id(); job < 6 * kt; job += waves) {
    const int j = job % 3, part = (job / 3) & 1, kh = (job / 6) * 16 + li;
    const float* row = vals + (j * 16 + li) * LV + lk;
    const float* wr = reinterpret_cast<const float*>(ws + min(kh, Kh - 1) * row_ld(N2)) + part;
    floatx4 acc = zero4();
    constexpr int U = 8;
    for (int ks = 0; ks < nk; ks += U) {
      float a[U];
      float t[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        a[u] = row[4 * min(ks + u, nk - 1)];
        t[u] = wr[2 * min(4 * (ks + u) + lk, N2 - 1)];
        if (ks + u >= nk) a[u] = 0.f;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u], t[u], acc, 0, 0, 0);
    }
    if (kh < Kh) {
#pragma unroll
      for (int r = 0; r < 4; ++r) store(j, 4 * lk + r, 2 * kh + part, acc[r]);
    }
  }
}

__device__ __forceinline__ float central_diff(const float* __restrict__ m, int x0, int x1, int x2,
                                              int N0, int N1, int N2, int axis) {
  if (axis == 0) {
    int p = (x0 + 1 == N0) ? 0 : x0 + 1, q = (x0 == 0) ? N0 - 1 : x0 - 1;
    return (m[((unsigned)p * N1 + x1) * N2 + x2] - m[((unsigned)q * N1 + x1) * N2 + x2]) * (0.5f * N0);
  }
  if (axis == 1) {
    int p = (x1 + 1 == N1) ? 0 : x1 + 1, q = (x1 == 0) ? N1 - 1 : x1 - 1;
    return (m[((unsigned)x0 * N1 + p) * N2 + x2] - m[((unsigned)x0 * N1 + q) * N2 + x2]) * (0.5f * N1);
  }
  int p = (x2 + 1 == N2) ? 0 : x2 + 1, q = (x2 == 0) ? N2 - 1 : x2 - 1;
  return (m[((unsigned)x0 * N1 + x1) * N2 + p] - m[((unsigned)x0 * N1 + x1) * N2 + q]) * (0.5f * N2);
}

// ------------------- image-term source and forward stage 2 (N grid)
// s_j = coef * [(a - b) * d_j m + res * d_j a] (periodic central
// differences; b and res may be null) at the points of 16 x1 rows of plane x0, contracted
// over x2: s1[j][x0][x1][kh].
template <class G>
__global__ void __launch_bounds__(kSrcThreads) k_src_fwd2(const float* __restrict__ a,
                                                  const float* __restrict__ b,
                                                  const float* __restrict__ res,
                                                  const float* __restrict__ m, float coef,
                                                  float2* __restrict__ s1, Twiddles tw, G gs) {
  extern __shared__ float shs[];
  const int N0 = gs.N0(), N1 = gs.N1(), N2 = gs.N2(), Kh = gs.Kh();
  const uint3 bk = xcd_block3<false>();
  const int x0 = bk.y, x1b = 16 * bk.x;
  const int rv = min(16, N1 - x1b);
  const int LV = tile_ld(N2), L4 = (N2 + 3) & ~3;
  float* vals = shs;  // [3][16][LV]
  float2* ws = reinterpret_cast<float2*>(shs + 48 * LV);
  stage_fwd2(ws, tw.fwd2, N2, Kh);
  // Two points per iteration, every load of a point unconditional (a load under a
  // branch waits for every load in flight): points past the tile repeat one.
  const float* bb = b ? b : a;
#pragma unroll 2
  for (int p = threadIdx.x; p < 16 * L4; p += kSrcThreads) {
    const int r = p / L4, x2 = p - r * L4;
    const int x1 = min(x1b + r, N1 - 1), xc = min(x2, N2 - 1);
    const unsigned gi = ((unsigned)x0 * N1 + x1) * N2 + xc;
    const float av = a[gi], bv = bb[gi];
    float v0 = central_diff(m, x0, x1, xc, N0, N1, N2, 0), v1 = central_diff(m, x0, x1, xc, N0, N1, N2, 1),
          v2 = central_diff(m, x0, x1, xc, N0, N1, N2, 2);
    const float s = coef * (av - (b ? bv : 0.f));
    v0 = s * v0;
    v1 = s * v1;
    v2 = s * v2;
    if (res) {
      const float t = coef * res[gi];
      v0 = fmaf(t, central_diff(a, x0, x1, xc, N0, N1, N2, 0), v0);
      v1 = fmaf(t, central_diff(a, x0, x1, xc, N0, N1, N2, 1), v1);
      v2 = fmaf(t, central_diff(a, x0, x1, xc, N0, N1, N2, 2), v2);
    }
    if (r >= rv || x2 >= N2) v0 = v1 = v2 = 0.f;
    float* at = vals + r * LV + x2;
    at[0] = v0;
    at[16 * LV] = v1;
    at[32 * LV] = v2;
  }
  __syncthreads();
  fwd2_tile(vals, ws, N2, Kh, kSrcThreads / 64, [&](int j, int r, int e, float v) {
    if (r < rv) reinterpret_cast<float*>(s1)[(unsigned)(((j * N0 + x0) * N1 + x1b + r) * 2 * Kh + e)] = v;
  });
}


// ----------- exact adjoint of one semi-Lagrangian step, forward stage 2
// The reverse of m_{n+1}(x) = I[m_n](X(x)), X(x) = x - dt v(x) (voxels per
// axis, the departure point k_sl computes).  For the state adjoint lam of
// m_{n+1} (held as lam / coef): the transpose of the interpolation scatters
// lam(x) with the trilinear weights onto the eight corners of X(x) in
// lam_out (zero on entry), and the derivative with respect to
// the grid velocity, s_j(x) = -dt N_j coef lam(x) (d_j I[m_n])(X(x)) with the
// interpolant's exact slope in the cell of X, is contracted over x2 as in
// k_src_fwd2: s1[j][x0][x1][kh].
//
// One block per brick of 4 planes x 8 rows, which it passes in chunks of CW <= 64
// columns.  Eight global atomic adds a point bound this kernel, so the chunk's
// sums are gathered in LDS, in a window of 7 x 11 x (CW + 3) that starts one
// voxel below the chunk moved by the whole voxels of its centre's displacement:
// it takes every point whose displacement differs from the centre's by up to a
// voxel, the others add to lam_out directly: none of them where a step moves less
// than a voxel (the tested and measured problems), a quarter at 9 voxels a step, two
// thirds at 15 (gradient of 2 steps at 128^3 / band 32, 9 voxels a step: 1000 us with
// global atomics, 483 so; of one step of 15 at 64^3 / band 16: 267, 184).  Then each entry that was touched
// is added to lam_out once, in runs along x2.  (The window is in FP64:
// ds_add_f64 takes 10 cycles a wave, ds_add_f32 196.)  Stage 2 keeps its sums in
// the registers of the wave that owns them, over the chunks, and its table for a
// chunk is on its way while the points are sampled (16 bytes, two columns, a
// lane: the even columns of 8 are one k-step, the odd ones the next).  At most 67 KB of LDS: two
// blocks a CU, so that one samples while the other multiplies.  At 160x192x160 /
// band 32: 250 us with global atomics, 240 with an FP32 window, 79 so, of which
// about 12 go to the products, 8 to the adds to lam_out and 14 to those in
// LDS; the rest is the points' arithmetic (about 200 vector instructions each).
constexpr int kAdjPlanes = 4, kAdjRows = 8, kAdjCols = 64, kAdjThreads = 512;
constexpr int kAdjW0 = kAdjPlanes + 3, kAdjW1 = kAdjRows + 3;
__host__ __device__ inline int adj_cols(int N2) {
  const int n = (N2 + kAdjCols - 1) / kAdjCols;
  return ((N2 + n - 1) / n + 7) & ~7;
}
template <int KT, class G>
__global__ void __launch_bounds__(kAdjThreads, 4) k_adj_src_fwd2(const float* __restrict__ lam,
                                                                 const float* __restrict__ m,
                                                                 const float* __restrict__ vel,
                                                                 float* __restrict__ lam_out, float coef, float dt,
                                                                 float2* __restrict__ s1, Twiddles tw, G gs) {
  extern __shared__ float shs[];
  constexpr int P = kAdjPlanes, R = kAdjRows, W0 = kAdjW0, W1 = kAdjW1, KS = kAdjCols / 8;
  constexpr int kPoints = P * R * kAdjCols / kAdjThreads;
  const int N0 = gs.N0(), N1 = gs.N1(), N2 = gs.N2(), Kh = gs.Kh();
  const unsigned nN = (unsigned)N0 * N1 * N2;
  const uint3 bk = xcd_block3<false>();
  const int x1b = R * bk.x, x0b = P * bk.y;
  const int CW = adj_cols(N2), LV = CW + 2, W2 = CW + 3;
  float* vals = shs;                                          // [2 plane pairs][3][16 rows][LV]
  double* win = reinterpret_cast<double*>(shs + 96 * LV);     // [W0][W1][W2]
  const int wave = wave_id(), lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  // stage 2: wave w < 6 owns (plane pair w / 3, field w % 3), all kh
  const int pp = wave / 3, j = wave % 3;
  floatx4 re[KT], im[KT];
#pragma unroll
  for (int q = 0; q < KT; ++q) re[q] = im[q] = zero4();
  for (int c = 0; c < N2; c += CW) {
    const int nc = min(CW, N2 - c);
    float4 t[KT][KS];
    auto table = [&](int q) {
      const float2* wr = tw.fwd2 + (unsigned)(min(16 * q + li, Kh - 1) * N2);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        t[q][ks] = ldu4(reinterpret_cast<const float*>(wr + min(c + 8 * ks + 2 * lk, N2 - 2)));
    };
    if (wave < 6) table(0);
    for (int i = threadIdx.x; i < W0 * W1 * W2; i += kAdjThreads) win[i] = 0.0;
    int o0, o1, o2;
    {
      const unsigned gc = ((unsigned)min(x0b + P / 2, N0 - 1) * N1 + min(x1b + R / 2, N1 - 1)) * N2 + c + nc / 2;
      const float d0 = -dt * vel[gc] * (float)N0, d1 = -dt * vel[nN + gc] * (float)N1,
                  d2 = -dt * vel[2 * nN + gc] * (float)N2;
      o0 = x0b - 1 + (fabsf(d0) < 1e6f ? (int)floorf(d0) : 0);
      o1 = x1b - 1 + (fabsf(d1) < 1e6f ? (int)floorf(d1) : 0);
      o2 = c - 1 + (fabsf(d2) < 1e6f ? (int)floorf(d2) : 0);
    }
    __syncthreads();
#pragma unroll 2
    for (int u = 0; u < kPoints; ++u) {
      const int p = threadIdx.x + u * kAdjThreads;
      const int r = p / CW, y = p - r * CW;
      if (r >= P * R) break;
      const int x0 = x0b + r / R, x1 = x1b + r % R, x2 = c + y;
      float g0 = 0.f, g1 = 0.f, g2 = 0.f;
      if (x0 < N0 && x1 < N1 && x2 < N2) {
        const unsigned gi = ((unsigned)x0 * N1 + x1) * N2 + x2;
        const Cell cl = cell_at((float)x0 - dt * vel[gi] * (float)N0, (float)x1 - dt * vel[nN + gi] * (float)N1,
                                (float)x2 - dt * vel[2 * nN + gi] * (float)N2, x0, x1, x2, gs);
        float v[8], d0, d1, d2;
        corners(m, cl, v, gs);
        slopes8(v, cl, &d0, &d1, &d2);
        const float l = lam[gi];
        const float s = -dt * coef * l;
        g0 = s * (float)N0 * d0;
        g1 = s * (float)N1 * d1;
        g2 = s * (float)N2 * d2;
        // transpose of the interpolation
        const float w0 = cl.w0, w1 = cl.w1, w2 = cl.w2, u0 = 1.f - w0, u1 = 1.f - w1, u2 = 1.f - w2;
        const unsigned j0 = (unsigned)cl.f0 - (unsigned)o0, j1 = (unsigned)cl.f1 - (unsigned)o1,
                       j2 = (unsigned)cl.f2 - (unsigned)o2;
        const float a[4] = {l * u0 * u1, l * u0 * w1, l * w0 * u1, l * w0 * w1};
        if (j0 < (unsigned)(W0 - 1) && j1 < (unsigned)(W1 - 1) && j2 < (unsigned)(W2 - 1)) {
          double* q = win + (j0 * W1 + j1) * W2 + j2;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            double* row = q + ((e >> 1) * W1 + (e & 1)) * W2;
            atomicAdd(row, (double)(a[e] * u2));
            atomicAdd(row + 1, (double)(a[e] * w2));
          }
        } else {
          const int b2 = (cl.a2 + 1 == N2) ? 0 : cl.a2 + 1;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            atomicAdd(lam_out + (cl.r[e] + cl.a2), a[e] * u2);
            atomicAdd(lam_out + (cl.r[e] + b2), a[e] * w2);
          }
        }
      }
      float* at = vals + ((r / 16) * 48 + r % 16) * LV + y;
      at[0] = g0;
      at[16 * LV] = g1;
      at[32 * LV] = g2;
    }
    __syncthreads();
    if (wave < 6) {
      const float* row = vals + ((pp * 3 + j) * 16 + li) * LV + 2 * lk;
      if constexpr (KT > 1) table(1);
#pragma unroll
      for (int q = 0; q < KT; ++q) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          if (8 * ks >= CW) break;
          const float2 a = *reinterpret_cast<const float2*>(row + 8 * ks);
          const bool last = c + 8 * ks + 2 * lk > N2 - 2;  // the load began at N2 - 2
          const float tx = last ? t[q][ks].z : t[q][ks].x, ty = last ? t[q][ks].w : t[q][ks].y;
          re[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, tx, re[q], 0, 0, 0);
          im[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, ty, im[q], 0, 0, 0);
          re[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, t[q][ks].z, re[q], 0, 0, 0);
          im[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, t[q][ks].w, im[q], 0, 0, 0);
        }
      }
    }
    for (int row = wave; row < W0 * W1; row += kAdjThreads / 64) {
      const int a0 = wrap(o0 + row / W1, N0), a1 = wrap(o1 + row % W1, N1);
      float* out = lam_out + (size_t)((unsigned)(a0 * N1 + a1) * N2);
      for (int y = lane; y < W2; y += 64) {
        const float v = (float)win[row * W2 + y];
        if (v != 0.f) atomicAdd(out + wrap(o2 + y, N2), v);
      }
    }
    __syncthreads();
  }
  if (wave >= 6) return;
#pragma unroll
  for (int q = 0; q < KT; ++q) {
    const int kh = 16 * q + li;
    if (kh >= Kh) continue;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 16 * pp + 4 * lk + r, x0 = x0b + row / R, x1 = x1b + row % R;
      if (x0 < N0 && x1 < N1) s1[(unsigned)(((j * N0 + x0) * N1 + x1) * Kh + kh)] = make_float2(re[q][r], im[q][r]);
    }
  }
}

// At phi(x) = x + u(x) (voxel coordinates x_j + N_j u_j) the periodic
// trilinear interpolation of I0, of its central-difference gradient G and
// (full Newton) of its central-difference Hessian H gives m, g and h.
// op 0: s_j = coef (m - I1) g_j.  op 1: s_j = coef (g . du) g_j
// [+ coef res (h du)_j when res is set].  Then forward stage 2 of the three
// sources like k_src_fwd2.
template <class G>
__global__ void __launch_bounds__(kSrcThreads) k_rho_fwd2(RhoArgs a, float2* __restrict__ s1, Twiddles tw, G gs) {
  extern __shared__ float shs[];
  const int N0 = gs.N0(), N1 = gs.N1(), N2 = gs.N2(), Kh = gs.Kh();
  const long long nN = (long long)N0 * N1 * N2;
  const uint3 bk = xcd_block3<false>();
  const int x0 = bk.y, x1b = 16 * bk.x;
  const int rv = min(16, N1 - x1b);
  const int LV = tile_ld(N2), L4 = (N2 + 3) & ~3;
  float* vals = shs;  // [3][16][LV]
  float2* ws = reinterpret_cast<float2*>(shs + 48 * LV);
  stage_fwd2(ws, tw.fwd2, N2, Kh);
  // two points per iteration, so that two chains of dependent loads are in flight
#pragma unroll 2
  for (int p = threadIdx.x; p < 16 * L4; p += blockDim.x) {
    const int r = p / L4, x2 = p % L4;
    const int x1 = x1b + r;
    float v0 = 0.f, v1 = 0.f, v2 = 0.f;
    if (r < rv && x2 < N2) {
      const unsigned gi = ((unsigned)x0 * N1 + x1) * N2 + x2;
      float X0 = (float)x0 + a.u[gi] * (float)N0;
      float X1 = (float)x1 + a.u[nN + gi] * (float)N1;
      float X2 = (float)x2 + a.u[2 * nN + gi] * (float)N2;
      // a non-finite displacement must not turn into an out-of-range index
      if (!isfinite(X0)) X0 = (float)x0;
      if (!isfinite(X1)) X1 = (float)x1;
      if (!isfinite(X2)) X2 = (float)x2;
      const float f0 = floorf(X0), f1 = floorf(X1), f2 = floorf(X2);
      const float w0 = X0 - f0, w1 = X1 - f1, w2 = X2 - f2;
      const int a0 = wrap((int)f0, N0), a1 = wrap((int)f1, N1), a2 = wrap((int)f2, N2);
      const int b0 = (a0 + 1 == N0) ? 0 : a0 + 1;
      const int b1 = (a1 + 1 == N1) ? 0 : a1 + 1;
      const int b2 = (a2 + 1 == N2) ? 0 : a2 + 1;
      const long long r00 = ((long long)a0 * N1 + a1) * N2, r01 = ((long long)a0 * N1 + b1) * N2;
      const long long r10 = ((long long)b0 * N1 + a1) * N2, r11 = ((long long)b0 * N1 + b1) * N2;
      // the four (or eight) channels of a point are one 16-byte load per corner
      auto lerp4 = [](float4 p, float4 q, float w) {
        return make_float4(p.x + w * (q.x - p.x), p.y + w * (q.y - p.y), p.z + w * (q.z - p.z),
                           p.w + w * (q.w - p.w));
      };
      auto interp4 = [&](const float4* f, int stride) {
        const float4 c00 = lerp4(f[stride * (r00 + a2)], f[stride * (r00 + b2)], w2);
        const float4 c01 = lerp4(f[stride * (r01 + a2)], f[stride * (r01 + b2)], w2);
        const float4 c10 = lerp4(f[stride * (r10 + a2)], f[stride * (r10 + b2)], w2);
        const float4 c11 = lerp4(f[stride * (r11 + a2)], f[stride * (r11 + b2)], w2);
        return lerp4(lerp4(c00, c01, w1), lerp4(c10, c11, w1), w0);
      };
      const float4 ig = interp4(reinterpret_cast<const float4*>(a.G), 1);  // (I0, d0, d1, d2)
      const float g0 = ig.y, g1 = ig.z, g2 = ig.w;
      if (a.op == 0) {
        const float l = a.coef * (ig.x - a.I1[gi]);
        v0 = l * g0;
        v1 = l * g1;
        v2 = l * g2;
      } else {
        const float du0 = a.du[gi], du1 = a.du[nN + gi], du2 = a.du[2 * nN + gi];
        const float l = a.coef * (g0 * du0 + g1 * du1 + g2 * du2);
        v0 = l * g0;
        v1 = l * g1;
        v2 = l * g2;
        if (a.res) {
          const float4 ha = interp4(reinterpret_cast<const float4*>(a.H), 2);      // (00, 01, 02, 11)
          const float4 hb = interp4(reinterpret_cast<const float4*>(a.H) + 1, 2);  // (12, 22, -, -)
          const float h00 = ha.x, h01 = ha.y, h02 = ha.z, h11 = ha.w, h12 = hb.x, h22 = hb.y;
          const float t = a.coef * a.res[gi];
          v0 = fmaf(t, h00 * du0 + h01 * du1 + h02 * du2, v0);
          v1 = fmaf(t, h01 * du0 + h11 * du1 + h12 * du2, v1);
          v2 = fmaf(t, h02 * du0 + h12 * du1 + h22 * du2, v2);
        }
      }
    }
    float* at = vals + r * LV + x2;
    at[0] = v0;
    at[16 * LV] = v1;
    at[32 * LV] = v2;
  }
  __syncthreads();
  fwd2_tile(vals, ws, N2, Kh, kSrcThreads / 64, [&](int j, int r, int e, float v) {
    if (r < rv) reinterpret_cast<float*>(s1)[(unsigned)(((j * N0 + x0) * N1 + x1b + r) * 2 * Kh + e)] = v;
  });
}


// ------------------------------------ forward stages 1 and 0 (x1, then x0)
// Complex sums over x of a 16 x 16 tile as matrix products, k-step ks holding
// x = 2 ks + h and the two parts of the product (lane lk = 2 h + part): per x
// first re w, then im w, the order of scalar code.  w is the table's row of this
// lane (w(k, x), k = lane % 16: read as it is, 16 bytes or two x a lane for four
// k-steps), v its data column (element lane % 16, the next x ld further).  The
// operands of the next 8 U x are on their way while the present ones are
// summed.  DataA: the data are the tile's rows, else its columns.  (A thread per
// output column and sums out of LDS: 20 and 17 us for stages 1 and 0 at
// 144x176x144 / band 24.)
template <bool DataA>
__device__ __forceinline__ void fwd_sum(const float2* __restrict__ w, const float2* __restrict__ v, unsigned ld, int N,
                                        floatx4* re, floatx4* im) {
  constexpr int U = 4;
  const int lk = (threadIdx.x & 63) >> 4, h = lk >> 1, part = lk & 1;
  struct Batch {
    float4 w[U];
    float2 v[U][4];
  } cur, nxt;
  auto load = [&](int x, Batch& b) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      b.w[u] = ldu4(reinterpret_cast<const float*>(w + min(x + 8 * u + 2 * lk, N - 2)));
#pragma unroll
      for (int k = 0; k < 4; ++k) b.v[u][k] = v[(unsigned)min(x + 8 * u + 2 * k + h, N - 1) * ld];
    }
  };
  floatx4 r = zero4(), i = zero4();
  load(0, cur);
  for (int x = 0; x < N; x += 8 * U) {
    if (x + 8 * U < N) load(x + 8 * U, nxt);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float4 q = cur.w[u];
      if (x + 8 * u + 2 * lk > N - 2) q = make_float4(q.z, q.w, q.z, q.w);  // the load began at N - 2
      float t[4], unused[4];
      pair_operands(q, t, unused);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const bool in = x + 8 * u + 2 * k + h < N;
        const float ex = in ? cur.v[u][k].x : 0.f, ey = in ? cur.v[u][k].y : 0.f;
        const float a = part ? -ey : ex, b = part ? ex : ey;
        if constexpr (DataA) {
          r = __builtin_amdgcn_mfma_f32_16x16x4f32(a, t[k], r, 0, 0, 0);
          i = __builtin_amdgcn_mfma_f32_16x16x4f32(b, t[k], i, 0, 0, 0);
        } else {
          r = __builtin_amdgcn_mfma_f32_16x16x4f32(t[k], a, r, 0, 0, 0);
          i = __builtin_amdgcn_mfma_f32_16x16x4f32(t[k], b, i, 0, 0, 0);
        }
      }
    }
    cur = nxt;
  }
  *re = r;
  *im = i;
}

// t[x0][kh][k1] = sum_x1 w(k1, x1) in[x0][x1][kh]: a wave forms one 16 x 16 tile
// (kh, k1) of one plane, a block four planes (which share the table's rows in L1).
__global__ void __launch_bounds__(256) k_fwd1(Fwd1Jobs jobs, const float2* __restrict__ tw, int G0, int G1, int K1,
                                              int Kh) {
  const Fwd1Job job = jobs.j[blockIdx.z];
  const int x0 = 4 * blockIdx.x + wave_id();
  if (x0 >= G0) return;
  const int t1 = (K1 + 15) / 16, k1b = 16 * (blockIdx.y % t1), khb = 16 * (blockIdx.y / t1);
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  floatx4 re, im;
  fwd_sum<true>(tw + (unsigned)(min(k1b + li, K1 - 1) * G1),
                job.in + (size_t)((unsigned)x0 * G1 * Kh) + min(khb + li, Kh - 1), Kh, G1, &re, &im);
  const int k1 = k1b + li;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int kh = khb + 4 * lk + r;
    if (kh < Kh && k1 < K1) job.out[(unsigned)((x0 * Kh + kh) * K1 + k1)] = make_float2(re[r], im[r]);
  }
}

// sum_x0 w(k0, x0) t[x0][c], c = kh K1 + k1, and the epilogue: a wave (a block)
// forms the 16 x 16 tile (k0, c) of one job.
__global__ void __launch_bounds__(64) k_fwd0(Fwd0Jobs jobs, const float2* __restrict__ tw,
                                             const float* __restrict__ Ksym, int G0, int K0, int K1, int Kh,
                                             float invG) {
  const Fwd0Job job = jobs.j[blockIdx.z];
  const int C = K1 * Kh, q0b = 16 * blockIdx.y;
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int c = 16 * blockIdx.x + li, cc = min(c, C - 1);
  const float2* w = tw + (unsigned)(min(q0b + li, K0 - 1) * G0);
  floatx4 are, aim, bre = zero4(), bim = zero4();
  fwd_sum<false>(w, job.a + cc, C, G0, &are, &aim);
  if (job.b) fwd_sum<false>(w, job.b + cc, C, G0, &bre, &bim);
  if (c >= C) return;
  const int q1 = c % K1, kh = c / K1;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int q0 = q0b + 4 * lk + r;
    if (q0 >= K0) continue;
    const unsigned idx = (unsigned)((kh * K0 + q0) * K1 + q1);
    const bool keep = q0 != K0 / 2 && q1 != K1 / 2;
    float2 v = make_float2(0.f, 0.f);
    if (keep) {
      if (job.base) v = job.base[idx];
      const float ks = Ksym[idx];
      const float sa = job.ca * invG * (job.syma ? ks : 1.f);
      v.x = fmaf(sa, are[r], v.x);
      v.y = fmaf(sa, aim[r], v.y);
      if (job.b) {
        const float sb = job.cb * invG * (job.symb ? ks : 1.f);
        v.x = fmaf(sb, bre[r], v.x);
        v.y = fmaf(sb, bim[r], v.y);
      }
      if (job.extra) {
        const float2 e = job.extra[idx];
        v.x = fmaf(job.ce, e.x, v.x);
        v.y = fmaf(job.ce, e.y, v.y);
      }
    }
    job.out[idx] = v;
    if (job.out2) {
      float2 v2 = make_float2(0.f, 0.f);
      if (keep) {
        const float s2 = job.ca * invG * Ksym[idx];
        v2.x = fmaf(s2, are[r], 0.f);
        v2.y = fmaf(s2, aim[r], 0.f);
      }
      job.out2[idx] = v2;
    }
  }
}

// LDS of a tile of fwd2_tile and its table (at most 50 + 66 KB)
constexpr size_t tile_bytes(int N2, int Kh) {
  return 48 * (size_t)tile_ld(N2) * sizeof(float) + (size_t)Kh * row_ld(N2) * sizeof(float2);
}
static_assert(tile_bytes(kMaxRow, kMaxBand / 2) <= kMaxLds);

// LDS of a brick of k_adj_src_fwd2 in chunks of CW columns (at most 67 KB, so that
// two fit a compute unit)
constexpr size_t adj_bytes(int CW) {
  return 96 * (size_t)(CW + 2) * sizeof(float) + (size_t)kAdjW0 * kAdjW1 * (CW + 3) * sizeof(double);
}
static_assert(2 * adj_bytes(kAdjCols) <= kMaxLds);

}  // namespace

hipError_t launch_fwd1(const Fwd1Jobs& jobs, int njobs, const float2* tw, int G0, int G1, int K1,
                       int Kh, hipStream_t st) {
  const dim3 grid(nblk(G0, 4), tiles16(K1) * tiles16(Kh), njobs);
  timer_work(KF_FWD1_GRID, njobs * 8.0 * G0 * Kh * (double)K1 * G1,
             njobs * 8.0 * ((double)G0 * G1 * Kh + (double)G0 * K1 * Kh));
  LAUNCH_TIMED(KF_FWD1_GRID, k_fwd1, grid, dim3(256), 0, st, jobs, tw, G0, G1, K1, Kh);
  return hipGetLastError();
}

hipError_t launch_fwd0(const Fwd0Jobs& jobs, int njobs, const float2* tw, const float* Ksym, int G0,
                       int K0, int K1, int Kh, float invG, hipStream_t st) {
  const dim3 grid(tiles16(K1 * Kh), tiles16(K0), njobs);
  {
    const double C = (double)K1 * Kh;
    double fl = 0, by = 0;
    for (int i = 0; i < njobs; ++i) {
      const Fwd0Job& j = jobs.j[i];
      int terms = 1 + (j.b != nullptr);
      fl += terms * 8.0 * K0 * C * G0;
      by += terms * 8.0 * G0 * C +
            8.0 * K0 * C * (1 + (j.base != nullptr) + (j.extra != nullptr) + (j.out2 != nullptr)) + 4.0 * K0 * C;
    }
    timer_work(KF_FWD0_GRID, fl, by);
  }
  LAUNCH_TIMED(KF_FWD0_GRID, k_fwd0, grid, dim3(64), 0, st, jobs, tw, Ksym, G0, K0, K1, Kh, invG);
  return hipGetLastError();
}

hipError_t launch_src_fwd2(const float* a, const float* b, const float* r, const float* m, float coef,
                           float2* s1, const Dims& d, const Twiddles& tw, hipStream_t st) {
  const dim3 grid(tiles16(d.N[1]), d.N[0]);
  const size_t shm = tile_bytes(d.N[2], d.Kh);
  {
    // gradient of m (6 flops / point / axis), the source, forward stage 2 of 3 fields
    const double nN = (double)d.nN;
    timer_work(KF_SRC, 3.0 * nN * d.Kh * 4.0 + (r ? 43.0 : 25.0) * nN,
               (b ? 12.0 : 8.0) * nN + (r ? 4.0 : 0.0) * nN + 3.0 * d.N[0] * (double)d.N[1] * d.Kh * 8.0);
  }
  hipError_t e = with_grid(d, [&](auto gs) {
    LAUNCH_TIMED(KF_SRC, (k_src_fwd2<decltype(gs)>), grid, dim3(kSrcThreads), shm, st, a, b, r, m, coef, s1, tw, gs);
    return hipGetLastError();
  });
  return e;
}

hipError_t launch_adj_src_fwd2(const float* lam, const float* m, const float* vel, float* lam_out, float coef,
                               float dt, float2* s1, const Dims& d, const Twiddles& tw, hipStream_t st) {
  const dim3 grid(nblk(d.N[1], kAdjRows), nblk(d.N[0], kAdjPlanes));
  const int CW = adj_cols(d.N[2]);
  const size_t shm = adj_bytes(CW);
  {
    // departure point, 8 gathers, slopes, 8 scattered weights, forward stage 2 of 3 fields
    const double nN = (double)d.nN;
    timer_work(KF_SRC, 3.0 * nN * d.Kh * 4.0 + 80.0 * nN,
               (4.0 + 12.0 + 4.0 + 8.0 * 4.0) * nN + 3.0 * d.N[0] * (double)d.N[1] * d.Kh * 8.0);
  }
  return with_grid(d, [&](auto gs) {
    using G = decltype(gs);
    if (d.Kh <= 16)
      LAUNCH_TIMED(KF_SRC, (k_adj_src_fwd2<1, G>), grid, dim3(kAdjThreads), shm, st, lam, m, vel, lam_out, coef, dt, s1,
                   tw, gs);
    else if constexpr (!G::kStatic)
      LAUNCH_TIMED(KF_SRC, (k_adj_src_fwd2<2, G>), grid, dim3(kAdjThreads), shm, st, lam, m, vel, lam_out, coef, dt, s1,
                   tw, gs);
    return hipGetLastError();
  });
}

hipError_t launch_rho_fwd2(const RhoArgs& a, float2* s1, const Dims& d, const Twiddles& tw, hipStream_t st) {
  const dim3 grid(tiles16(d.N[1]), d.N[0]);
  const size_t shm = tile_bytes(d.N[2], d.Kh);
  {
    // trilinear interpolation of 4 (op 0), 3 or 9 (op 1) fields, the source,
    // forward stage 2 of 3 fields; point reads u (3) and I1 | du (3), res
    const double nN = (double)d.nN;
    const bool full = a.op == 1 && a.res;
    const double nf = a.op == 0 ? 4.0 : (full ? 9.0 : 3.0);
    const double rd = a.op == 0 ? 4.0 : (full ? 7.0 : 6.0);
    timer_work(KF_SRC, 3.0 * nN * d.Kh * 4.0 + (nf * 14.0 + (full ? 30.0 : 12.0)) * nN,
               (nf + rd) * 4.0 * nN + 3.0 * d.N[0] * (double)d.N[1] * d.Kh * 8.0);
  }
  hipError_t e = with_grid(d, [&](auto gs) {
    LAUNCH_TIMED(KF_SRC, (k_rho_fwd2<decltype(gs)>), grid, dim3(kSrcThreads), shm, st, a, s1, tw, gs);
    return hipGetLastError();
  });
  return e;
}

}  // namespace lddmm
