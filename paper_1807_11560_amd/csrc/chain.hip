// Kernels of the shapes without instantiated ones: the transforms between the
// band and a grid as chained matrix products at any size (see mfma.h), and the
// tables of all shapes.
#include "mfma.h"

#include <math.h>

#include <algorithm>
#include <type_traits>

#include "launch.h"
#include "sample.h"
#include "shapes.h"

namespace lddmm {

// ------------------------------------------------------------------ tables
__device__ __forceinline__ double2 unit_wave(int k, int x, int G) {
  long long r = ((long long)k * x) % G;
  if (r < 0) r += G;
  double s, c;
  sincospi(2.0 * (double)r / (double)G, &s, &c);
  return make_double2(c, s);
}

// exp(2 pi i k x / G) (v = 1: times 2 pi i k) of the full axis's slot q, zero
// on the slot -K/2, or with `half` of frequency q with weight 1 or 2.
__device__ __forceinline__ float2 inverse_entry(int q, int K, int x, int G, int v, bool half) {
  if (!half && q == K / 2) return make_float2(0.f, 0.f);
  const int k = half ? q : (q < K / 2 ? q : q - K);
  const double2 e = unit_wave(k, x, G);
  double re = e.x, im = e.y;
  if (v == 1) {
    const double w = 2.0 * M_PI * (double)k, nre = -w * im, nim = w * re;
    re = nre;
    im = nim;
  }
  if (half && q > 0) {
    re *= 2.0;
    im *= 2.0;
  }
  return make_float2((float)re, (float)im);
}
__device__ __forceinline__ float2 forward_entry(int q, int K, int x, int G, bool half) {
  if (!half && q == K / 2) return make_float2(0.f, 0.f);
  const double2 e = unit_wave(half ? q : (q < K / 2 ? q : q - K), x, G);
  return make_float2((float)e.x, (float)-e.y);
}

// Every table of a problem in one launch (17 launches of 2 us before, and the
// gaps between them: 30 to 50 us of each call that shoots): block row y works on
// job y.
// Plain kinds: inverse [2][G][K], inverse half [2][G][K/2], forward [K][G],
// forward half [K/2][G].
__global__ void k_tables(TableJobs jobs) {
  const TableJob& j = jobs.j[blockIdx.y];
  const int K = j.K, G = j.G;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < j.total; i += gridDim.x * blockDim.x) {
    switch (j.kind) {
      case TAB_INV:
        static_cast<float2*>(j.dst)[i] = inverse_entry(i % K, K, (i / K) % G, G, i / (G * K), false);
        break;
      case TAB_FWD:
      case TAB_FWD_HALF:
        static_cast<float2*>(j.dst)[i] = forward_entry(i / G, K, i % G, G, j.kind == TAB_FWD_HALF);
        break;
      case TAB_ROW_INV:
      case TAB_ROW_INV_HALF:
      case TAB_ROW_INV_POS:
      case TAB_ROW_INV_HALF_POS: {
        const int KT = (K + 15) / 16, GT = (G + 15) / 16;
        const int lane = (i >> 2) & 63, rest = i >> 8;
        const int q = 16 * (rest % KT) + 4 * (i & 3) + (lane >> 4), part = (rest / KT) % 2;
        const int x = 16 * ((rest / (2 * KT)) % GT) + (lane & 15);
        float2 w = make_float2(0.f, 0.f);
        if (q < K && x < G) w = inverse_entry(q, K, x, G, rest / (2 * KT * GT),
                                              j.kind == TAB_ROW_INV_HALF || j.kind == TAB_ROW_INV_HALF_POS);
        const bool neg = j.kind == TAB_ROW_INV || j.kind == TAB_ROW_INV_HALF;
        static_cast<float*>(j.dst)[i] = part ? (neg ? -w.y : w.y) : w.x;
        break;
      }
      case TAB_PAIR_INV:
      case TAB_PAIR_INV_HALF:
      case TAB_PAIR_FWD: {  // one float per lane and k-step
        const int lane = (i >> 2) & 63, rest = i >> 8, li = lane & 15, lk = lane >> 4;
        const int D = j.kind == TAB_PAIR_FWD ? G : K, JT = (D + 7) / 8;
        const int at = 2 * (4 * (rest % JT) + (i & 3)) + (lk >> 1), tile = rest / JT;
        float2 w = make_float2(0.f, 0.f);
        if (j.kind == TAB_PAIR_FWD) {
          if (16 * tile + li < K && at < G) w = forward_entry(16 * tile + li, K, at, G, false);
        } else {
          const int GT = (G + 15) / 16, x = 16 * (tile % GT) + li;
          if (at < K && x < G) w = inverse_entry(at, K, x, G, tile / GT, j.kind == TAB_PAIR_INV_HALF);
          if (j.kind == TAB_PAIR_INV_HALF) w.y = -w.y;
        }
        static_cast<float*>(j.dst)[i] = (lk & 1) ? w.y : w.x;
        break;
      }
      case TAB_COL1: {  // [x][Kp]
        const int Kp = (K + 15) & ~15, k = i % Kp;
        static_cast<float2*>(j.dst)[i] = k < K ? forward_entry(k, K, i / Kp, G, false) : make_float2(0.f, 0.f);
        break;
      }
      case TAB_COL0:  // [Kp][x]
        static_cast<float2*>(j.dst)[i] = i / G < K ? forward_entry(i / G, K, i % G, G, false) : make_float2(0.f, 0.f);
        break;
      case TAB_COL0_INV: {  // [2][Mp][K]
        const int Mp = (G + 15) & ~15, x = (i / K) % Mp;
        static_cast<float2*>(j.dst)[i] =
            x < G ? inverse_entry(i % K, K, x, G, i / (Mp * K), false) : make_float2(0.f, 0.f);
        break;
      }
      case TAB_SYMBOLS: {  // band layout [Kh][K0][K1]
        const float2 lk = band_symbols((i / G) % K, i % G, i / (K * G), K, G, j.s, j.alpha);
        static_cast<float*>(j.dst)[i] = lk.x;
        static_cast<float*>(j.dst2)[i] = lk.y;
        break;
      }
      default:
        static_cast<unsigned*>(j.dst)[i] = 0u;
    }
  }
}

hipError_t launch_tables(const TableJobs& jobs, int njobs, hipStream_t st) {
  int most = 1;
  for (int i = 0; i < njobs; ++i) most = std::max(most, jobs.j[i].total);
  hipLaunchKernelGGL(k_tables, dim3(std::min(nblk(most, 256), 64u), njobs), dim3(256), 0, st, jobs);
  return hipGetLastError();
}

// ---------------------------------------------- synthesis on the padded grid
// One wave per (x0 plane, new field (group, component), 16 x1): inverse stages
// 1 (k1 -> x1) and 2 (half spectrum -> real x2) of the variants value, d/dx1
// (stage-1 derivative table), d/dx0 (derivative stage-0 input) and d/dx2
// (stage-2 derivative table), both sums in "rows" order.  Stage 1 forms
// T2[kh][x1], rows named kh = 16 kt + 4 r + lk, the A operand [x1][kh] of stage
// 2, whose result has columns x2: 16 lanes store 16 consecutive points of
// (value, d0, d1, d2), 256 bytes.  Nothing goes through LDS and no wave waits
// for another; a lane's part of the stage-0 input (KQ groups of 16 k1) is
// loaded at once and used for both parts.
// Bound by the matrix cores at large bands (band 64, M = 96: 768 products a
// wave, 35 us of them in a launch, 85 MB stored): 324 us with the operands staged
// through LDS one compute unit at a time, 73 us here (86 with an 8-byte load per
// operand, whose 16-lane quarters touch 16 rows and take 64 cycles of the address
// unit: now one 16-byte load for two k-steps); band 40: 41 -> 25 us.
template <int KT, int KQ, bool BF3>
__global__ void __launch_bounds__(256, BF3 ? 3 : 4) k_synth_chain(SynthArgs a, const float4* __restrict__ fr1,
                                                                  const float4* __restrict__ fr2, BandDyn sh) {
  using O = Op<BF3>;
  const int M0 = sh.M0(), M1 = sh.M1(), M2 = sh.M2(), K1 = sh.K1(), Kh = sh.Kh();
  const int X1T = (M1 + 15) / 16, X2T = (M2 + 15) / 16;
  const int wave = wave_id(), lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int g = blockIdx.y / 3, c = blockIdx.y % 3;
  const int task = blockIdx.x * 4 + wave;
  if (task >= M0 * X1T) return;
  const int x0 = task / X1T, x1t = task % X1T;
  const float2* src = a.t1[g] + (size_t)c * 2 * M0 * K1 * Kh;
  float t2[3][KT][2][4];  // variant (value, d1, d0), kh tile, re / im, register
#pragma unroll
  for (int kt = 0; kt < KT; ++kt) {
    // rows past Kh and k1 past K1 repeat the last one: they meet zero table entries
    const int kh = min(16 * kt + 4 * (li & 3) + (li >> 2), Kh - 1);
    // stage-0 input vs (plain, then d0) against the stage-1 tables (plain and
    // derivative, or plain alone); the table of the next group arrives during
    // this group's products
    auto stage1 = [&](auto VS) {
      constexpr int vs = decltype(VS)::value, NV = vs ? 1 : 2;
      const float2* plane = src + ((size_t)vs * M0 + x0) * Kh * K1;
      const unsigned row = kh * K1;
      asm volatile("" ::: "memory");  // one input's loads at a time: their registers bound the waves
      __builtin_amdgcn_sched_barrier(0);
      float2 t[KQ][4];
#pragma unroll
      for (int q = 0; q < KQ; ++q)
#pragma unroll
        for (int u = 0; u < 4; u += 2) {
          const unsigned k = 16 * q + 4 * u + 2 * lk;  // only the last group can pass K1
          const floatx4 v = *reinterpret_cast<const floatx4*>(plane + (row + (q == KQ - 1 ? min(k, (unsigned)K1 - 2) : k)));
          t[q][u] = make_float2(v.x, v.y);
          t[q][u + 1] = make_float2(v.z, v.w);
        }
      float4 tb[NV], nx[NV];
      auto table = [&](int pq, float4 (&w)[NV]) {
#pragma unroll
        for (int v = 0; v < NV; ++v) w[v] = (fr1 + (((size_t)v * X1T + x1t) * 2 * KQ + pq) * 64)[lane];
      };
      table(0, tb);
      floatx4 acc[NV][2];
#pragma unroll
      for (int v = 0; v < NV; ++v) acc[v][0] = acc[v][1] = zero4();
#pragma unroll
      for (int pq = 0; pq < 2 * KQ; ++pq) {
        const int part = pq / KQ, q = pq % KQ;
        if (pq + 1 < 2 * KQ) table(pq + 1, nx);
        if (part == 0) {
#pragma unroll
          for (int u = 0; u < 4; u += 2) {
            swap_quarters(t[q][u].x, t[q][u + 1].x);
            swap_quarters(t[q][u].y, t[q][u + 1].y);
          }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float2 p = t[q][u];
          const typename O::T pr = O::a(part ? p.y : p.x), pi = O::a(part ? -p.x : p.y);
#pragma unroll
          for (int v = 0; v < NV; ++v) {
            const typename O::T b = O::b(elem(tb[v], u));
            acc[v][0] = O::mma(pr, b, acc[v][0]);
            acc[v][1] = O::mma(pi, b, acc[v][1]);
          }
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) tb[v] = nx[v];
        __builtin_amdgcn_sched_barrier(0);  // later tables are not loaded yet: their registers bound the waves
      }
#pragma unroll
      for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int r = 0; r < 4; ++r) t2[vs ? 2 : v][kt][q][r] = acc[v][q][r];
    };
    stage1(std::integral_constant<int, 0>{});
    stage1(std::integral_constant<int, 1>{});
  }
  const long long nM = (long long)M0 * M1 * M2;
  float* out = a.dst[g] + ((size_t)c * nM + (size_t)x0 * M1 * M2) * 4;
  float4 tb[2][KT], nx[2][KT];
  auto table = [&](int s, float4 (&w)[2][KT]) {  // s = 2 x2t + part
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) w[v][kt] = (fr2 + (((size_t)v * X2T * 2 + s) * KT + kt) * 64)[lane];
  };
  table(0, tb);
  for (int x2t = 0; x2t < X2T; ++x2t) {
    floatx4 f[4];  // value, d0, d1, d2
#pragma unroll
    for (int v = 0; v < 4; ++v) f[v] = zero4();
#pragma unroll
    for (int part = 0; part < 2; ++part) {
      table(min(2 * x2t + part + 1, 2 * X2T - 1), nx);  // arrives during this part's products
#pragma unroll
      for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const typename O::T b0 = O::b(elem(tb[0][kt], u)), b1 = O::b(elem(tb[1][kt], u));
          const typename O::T a0 = O::a(t2[0][kt][part][u]);
          f[0] = O::mma(a0, b0, f[0]);
          f[1] = O::mma(O::a(t2[2][kt][part][u]), b0, f[1]);
          f[2] = O::mma(O::a(t2[1][kt][part][u]), b0, f[2]);
          f[3] = O::mma(a0, b1, f[3]);
        }
#pragma unroll
      for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) tb[v][kt] = nx[v][kt];
    }
    const int x2 = 16 * x2t + li;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int x1 = 16 * x1t + 4 * lk + r;
      if (x1 < M1 && x2 < M2)
        reinterpret_cast<float4*>(out)[(unsigned)(x1 * M2 + x2)] = make_float4(f[0][r], f[1][r], f[2][r], f[3][r]);
    }
  }
}

// Calls f with a compile-time 1 .. N equal to n.
template <int N, class F>
static hipError_t with_int(int n, F&& f) {
  if constexpr (N > 1)
    if (n < N) return with_int<N - 1>(n, f);
  return f(std::integral_constant<int, N>{});
}

hipError_t launch_synth_chain(const SynthArgs& a, int nf, const Frags& fr, const Dims& d, hipStream_t st) {
  if (!fr.row1 || !fr.row2) return hipErrorInvalidValue;
  // four waves a block: one per SIMD, so that blocks pack by registers alone
  // (blocks of six waves left a compute unit with one block: 100 us at band 64)
  const dim3 grid(nblk((long long)d.M[0] * tiles16(d.M[1]), 4), nf), block(256);
  const BandDyn sh{d.K[0], d.K[1], d.Kh, d.M[0], d.M[1], d.M[2]};
  return with_int<2>(tiles16(d.Kh), [&](auto kt) {
    return with_int<4>(tiles16(d.K[1]), [&](auto kq) {
      constexpr int KT = decltype(kt)::value, KQ = decltype(kq)::value;
      if (d.prec)
        LAUNCH_TIMED(KF_SYNTH, (k_synth_chain<KT, KQ, true>), grid, block, 0, st, a, fr.row1, fr.row2, sh);
      else
        LAUNCH_TIMED(KF_SYNTH, (k_synth_chain<KT, KQ, false>), grid, block, 0, st, a, fr.row1, fr.row2, sh);
      return hipGetLastError();
    });
  });
}

// ------------------------------------------------ column step on the band side
// One block per (kh, job, 16 slots k1): forward stages 1 (x1 -> k1) and 0 (x0
// -> k0) of the job's one or two product fields, the band update, the next
// inverse stage 0 on the padded grid (value and d0 of out or L~ out) and on
// the image grid, every sum in "pairs" order, FP32 in both precisions.  Stage
// 1' takes the field straight from memory, 16 x0 per wave and step; its result,
// the update and the next stage's input meet in LDS (16 columns, 41 KB at
// band 64), the tables are read as 1 KB rows, the same for all blocks.  At small
// bands the launch is one chain of latencies: the update's values and the
// first tables of a phase are loaded before the phase begins, and the registers
// are kept under 128 so that two blocks share a compute unit (142: 85 us at band
// 64).  Against scalar sums out of LDS: 243 -> 47 us at band 64, 34 -> 19 us at
// band 40, 13.1 -> 9.4 us at band 24x20x20 (with two loads for four k-steps of the
// field 52, 20 and 10).
template <int GC>       // groups of four k-steps per load; the next ones are in flight
struct ColTab {         // a fragment table being walked: w holds groups j .. j + GC - 1
  const float4* p;
  int J;
  float4 w[GC];
  __device__ __forceinline__ void open(const float4* tab, int n) {
    p = tab;
    J = n;
    load(0, w);
  }
  __device__ __forceinline__ void load(int j, float4 (&o)[GC]) const {
#pragma unroll
    for (int q = 0; q < GC; ++q) o[q] = (p + (size_t)min(j + q, J - 1) * 64)[threadIdx.x & 63];
  }
};

template <int NW>
__global__ void __launch_bounds__(64 * NW, 4) k_column_chain(ColJobs jobs, Frags fM, Frags fN,
                                                          const float* __restrict__ Lsym,
                                                          const float* __restrict__ Ksym, BandDyn sh, float invG) {
  extern __shared__ float2 cl[];
  const int M0 = sh.M0(), M1 = sh.M1(), K0 = sh.K0(), K1 = sh.K1(), Kh = sh.Kh();
  const int M0p = (M0 + 15) & ~15, K0p = (K0 + 15) & ~15;
  const int XT = M0p / 16, K0T = K0p / 16;
  const int J0 = (K0 + 7) / 8, JM0 = (M0 + 7) / 8, JM1 = (M1 + 7) / 8;  // groups of four k-steps
  float2* s2 = cl;                   // [2][M0p][16]
  float2* fb = cl + 2 * M0p * 16;    // [K0p][16]   stage 0' of the second term
  float2* ob = fb;                   // [2][K0p][16] out, L~ out (after fb has been read)
  const uint3 lb = xcd_block3<true>();
  const ColJob& job = jobs.j[lb.y];
  const int kh = lb.x, kc = lb.z;
  const int wave = wave_id(), lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int h = lk >> 1, part = lk & 1;
  const unsigned neg = part ? 0x80000000u : 0u;
  const int nterm = job.a ? (job.b ? 2 : 1) : 0;
  const int k1 = 16 * kc + li;

  // stage 0' tile of this wave (K0 <= 64: at most four): the first term's on
  // waves 0 .. 3, the second's on the last four
  static_assert(NW >= 8, "a wave per stage-0' tile of both terms");
  const int t0 = wave < 4 ? 0 : 1, kt0 = t0 == 0 ? wave : NW - 1 - wave;
  const bool mine0 = kt0 < K0T && (t0 == 0 || nterm == 2);
  ColTab<4> f0;
  if (nterm) f0.open(fM.fwd0 + (size_t)min(kt0, K0T - 1) * JM0 * 64, JM0);
  // next inverse stage 0: padded-grid tiles (group, variant, 16 x0), then image-grid tiles
  const int npad = job.nt1 * 2 * XT, units = npad + (job.t1n ? (jobs.N0 + 15) / 16 : 0);
  auto unit_table = [&](int un) {
    return un < npad ? fM.inv0 + (size_t)((un / XT) % 2 * XT + un % XT) * J0 * 64
                     : fN.inv0 + (size_t)(un - npad) * J0 * 64;
  };

  // stage 1': s2[t][x0][k1] = sum_x1 fwd1[k1][x1] S[t][x0][x1]
  constexpr int kS = 2;
  for (int un = wave; un < nterm * XT; un += NW) {
    const int t = un / XT, xt = un % XT;
    const float2* plane = (t ? job.b : job.a) + (size_t)kh * M0 * M1;
    const unsigned row = min(16 * xt + li, M0 - 1) * M1;
    // four k-steps' values per 16-byte load (a row of odd length: its last pair
    // begins one earlier)
    auto load = [&](int j, float4 (&s)[kS]) {
#pragma unroll
      for (int q = 0; q < kS; ++q) {
        const int k = 8 * (j + q) + 2 * lk;
        s[q] = ldu4(reinterpret_cast<const float*>(plane + (row + min(k, M1 - 2))));
        if ((M1 & 1) && k > M1 - 2) {
          s[q].x = s[q].z;
          s[q].y = s[q].w;
        }
      }
    };
    ColTab<kS> f1;
    f1.open(fM.fwd1 + (size_t)kc * JM1 * 64, JM1);
    float4 s[kS], sn[kS];
    load(0, s);
    floatx4 re = zero4(), im = zero4();
    for (int j = 0; j < JM1; j += kS) {
      float4 wn[kS];
      f1.load(j + kS, wn);
      load(j + kS, sn);
#pragma unroll
      for (int q = 0; q < kS; ++q) {
        if (j + q >= JM1) break;
        float sr[4], si[4];
        pair_operands(s[q], sr, si);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float wi = elem(f1.w[q], u), wr = flip(wi, neg);
          re = Op<false>::mma(sr[u], wr, re);
          im = Op<false>::mma(si[u], wi, im);
        }
      }
#pragma unroll
      for (int q = 0; q < kS; ++q) {
        f1.w[q] = wn[q];
        s[q] = sn[q];
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) s2[((size_t)t * M0p + 16 * xt + 4 * lk + r) * 16 + li] = make_float2(re[r], im[r]);
  }
  // the update's values (unconditional loads: a job without an extra term reads
  // its base again, one without a base its first product at a valid index)
  float2 pb[4], pe[4];
  float pk[4], pl[4];
  {
    const float2* b = job.base ? job.base : job.a;
    const float2* x = job.extra ? job.extra : b;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const size_t idx = ((size_t)kh * K0 + min(16 * kt0 + 4 * lk + r, K0 - 1)) * K1 + min(k1, K1 - 1);
      pb[r] = b[idx];
      pe[r] = x[idx];
      pk[r] = Ksym[idx];
      pl[r] = Lsym[idx];
    }
  }
  ColTab<4> ft;
  ft.open(unit_table(min(wave, max(units - 1, 0))), J0);
  __syncthreads();

  // a tile of sum_k w(k) b(k), b in LDS [k][16], the table open at group 0
  auto product = [&](ColTab<4>& f, const float2* b, floatx4& re, floatx4& im) {
    for (int j = 0; j < f.J; j += 4) {
      float4 wn[4];
      f.load(j + 4, wn);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (j + q >= f.J) break;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float2 v = b[(size_t)(2 * (4 * (j + q) + u) + h) * 16 + li];
          const float wi = elem(f.w[q], u), wr = flip(wi, neg);
          re = Op<false>::mma(wr, part ? v.y : v.x, re);
          im = Op<false>::mma(wi, part ? v.x : v.y, im);
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) f.w[q] = wn[q];
    }
  };
  floatx4 fre = zero4(), fim = zero4();
  if (mine0 && nterm) product(f0, s2 + (size_t)t0 * M0p * 16, fre, fim);
  if (nterm == 2) {
    if (mine0 && t0 == 1) {
#pragma unroll
      for (int r = 0; r < 4; ++r) fb[(size_t)(16 * kt0 + 4 * lk + r) * 16 + li] = make_float2(fre[r], fim[r]);
    }
    __syncthreads();
  }
  float2 res[4];
  if (mine0 && t0 == 0) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int k0 = 16 * kt0 + 4 * lk + r;
      float2 v = make_float2(0.f, 0.f);
      if (k0 < K0 && k1 < K1) {
        if (k0 != K0 / 2 && k1 != K1 / 2) {
          if (job.base) v = pb[r];
          const float sa = job.ca * invG * (job.syma ? pk[r] : 1.f);
          if (nterm) {
            v.x = fmaf(sa, fre[r], v.x);
            v.y = fmaf(sa, fim[r], v.y);
          }
          if (nterm == 2) {
            const float2 o = fb[(size_t)k0 * 16 + li];
            const float sb = job.cb * invG * (job.symb ? pk[r] : 1.f);
            v.x = fmaf(sb, o.x, v.x);
            v.y = fmaf(sb, o.y, v.y);
          }
          if (job.extra) {
            v.x = fmaf(job.ce, pe[r].x, v.x);
            v.y = fmaf(job.ce, pe[r].y, v.y);
          }
        }
        if (job.out) job.out[((size_t)kh * K0 + k0) * K1 + k1] = v;
      }
      res[r] = v;
    }
  }
  if (units == 0) return;
  if (nterm == 2) __syncthreads();  // fb has been read
  if (mine0 && t0 == 0) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const size_t o = (size_t)(16 * kt0 + 4 * lk + r) * 16 + li;
      ob[o] = res[r];
      ob[(size_t)K0p * 16 + o] = make_float2(pl[r] * res[r].x, pl[r] * res[r].y);
    }
  }
  __syncthreads();
  for (int un = wave; un < units; un += NW) {
    const bool pad = un < npad;
    const int grp = pad ? un / (2 * XT) : 0, v = (un / XT) % 2, xt = pad ? un % XT : un - npad;
    const bool lsel = pad && (grp == 0 ? job.t1l[0] : job.t1l[1]);
    floatx4 re = zero4(), im = zero4();
    product(ft, ob + (lsel ? (size_t)K0p * 16 : 0), re, im);
    if (un + NW < units) ft.open(unit_table(un + NW), J0);
    if (k1 >= K1) continue;
    const int G0 = pad ? M0 : jobs.N0;
    float2* dst = pad ? (grp == 0 ? job.t1[0] : job.t1[1]) + (size_t)v * M0 * Kh * K1 : job.t1n;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int x0 = 16 * xt + 4 * lk + r;
      if (x0 < G0) dst[((size_t)x0 * Kh + kh) * K1 + k1] = make_float2(re[r], im[r]);
    }
  }
}

hipError_t launch_column_chain(const ColJobs& jobs, int njobs, const Dims& d, const Frags& frM, const Frags& frN,
                               const float* Lsym, const float* Ksym, float invG, hipStream_t st) {
  if (!frM.inv0 || !frM.fwd0 || !frM.fwd1 || !frN.inv0) return hipErrorInvalidValue;
  for (int i = 0; i < njobs; ++i)
    if ((!jobs.j[i].a && (!jobs.j[i].base || jobs.j[i].b)) || (jobs.j[i].a && !jobs.j[i].out)) return hipErrorInvalidValue;
  const int M0p = 16 * tiles16(d.M[0]), K0p = 16 * tiles16(d.K[0]);
  const size_t shm = (size_t)(2 * M0p + 2 * K0p) * 16 * sizeof(float2);
  static_assert((2 * kMaxPadded + 2 * kMaxBand) * 16 * sizeof(float2) <= kMaxLds);
  const dim3 grid(d.Kh, njobs, tiles16(d.K[1]));
  const BandDyn sh{d.K[0], d.K[1], d.Kh, d.M[0], d.M[1], d.M[2]};
  LAUNCH_TIMED(column_family(jobs), (k_column_chain<8>), grid, dim3(512), shm, st, jobs, frM, frN, Lsym, Ksym, sh, invG);
  return hipGetLastError();
}

// ------------------------------------------------------------- grid step
// One block of four waves per (x0, 16 x1): inverse stage 1 (k1 -> x1) of the
// three velocity components from their stage-0 output, one 16 x 16 (kh, x1)
// tile per wave and step, straight from memory; its result meets in LDS
// (3 Khp rows, 6 KB at 16 kh), and stage 2 (half spectrum -> real x2) gives each
// wave whole tiles of 16 x2 with all components, from which
//   the source is formed with four consecutive points of a row per lane (rows
//   x2 of the product, 16-byte loads and stores of m, dm and q; the loads are
//   issued before the products of the stage before them);
//   the velocity is stored, and the transport step done, with 16 consecutive
//   points of a row per 16 lanes (rows x1 of the product), so that the eight
//   gathers of a point meet those of its neighbours in a cache line.
// The transport from the registers saves reading the velocity back (12 of the 20
// bytes per point of a separate step) and, where no later call needs it,
// storing it.
// Measured, transport form: 180x210x180 / band 32, with the velocity stored, 125
// (grid step out of scalar sums 77, transport 48) -> 64 us; 160x192x160 without
// it 56 -> 35 us, of which the gathers are 10; source form 128^3 / band 64 117 ->
// 30 us alone.  Points along x2 per lane instead (16-byte stores, each
// gather over 16 rows) took the transport form from 35 to 51 us.
// Sums: with SEP the four real sums of a complex product are formed apart
// (order "rows", the instantiated grids), else in "pairs" order (all others,
// FP32 in both precisions).
template <class G>
__device__ __forceinline__ float4 row4(const float* p, int x2, G gs) {  // p[x2 .. x2 + 3], repeating inside the row past its end
  const int N2 = gs.N2();
  if (N2 % 4 == 0) return *reinterpret_cast<const float4*>(p + min(x2, N2 - 4));
  const int at = min(x2, N2 - 4), o = x2 - at;
  const float4 v = ldu4(p + at);
  if (o == 0) return v;
  return make_float4(o == 1 ? v.y : o == 2 ? v.z : v.w, o == 1 ? v.z : v.w, v.w, v.w);
}
template <class G>
__device__ __forceinline__ void put4(float* p, int x2, float4 v, G gs) {
  const int N2 = gs.N2();
  if (x2 >= N2) return;
  if (N2 % 4 == 0) {
    *reinterpret_cast<float4*>(p + x2) = v;
  } else if (x2 + 3 < N2) {
    f4_u4 u = {v.x, v.y, v.z, v.w};
    *reinterpret_cast<f4_u4*>(p + x2) = u;
  } else {
    p[x2] = v.x;
    if (x2 + 1 < N2) p[x2 + 1] = v.y;
    if (x2 + 2 < N2) p[x2 + 2] = v.z;
  }
}

template <int KT, int OP, bool SEP, bool BF3, class G>
__global__ void __launch_bounds__(256, 4) k_gridstep(GridStepArgs a, const float4* __restrict__ f1,
                                                     const float4* __restrict__ f2, G gs) {
  using O = Op<BF3>;
  constexpr int S = SEP ? 48 : 32;  // floats per kh row of the stage-1 result: (re | im) of 16 x1
  __shared__ float t2[3 * 16 * KT * S];
  const int N0 = gs.N0(), N1 = gs.N1(), N2 = gs.N2(), K1 = gs.K1(), Kh = gs.Kh();
  const int X2T = (N2 + 15) / 16, KQ = (K1 + 15) / 16, J1 = (K1 + 7) / 8, J2 = (Kh + 7) / 8;
  // the row tiles of one plane read the same stage-0 input: one XCD each
  const uint3 lb = xcd_block3<false>();
  const int x0 = lb.y, x1t = lb.x;
  const int wave = wave_id(), lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int h = lk >> 1, part = lk & 1;
  const unsigned neg = part ? 0x80000000u : 0u;
  const int x1 = 16 * x1t + li, x1c = min(x1, N1 - 1);  // of the source's points

  struct Near { float4 c, p0, m0, p1, m1, dm; float lo, hi; } near, nxt;
  auto fetch = [&](int x2t, Near& o) {
    const size_t NN = (size_t)N1 * N2;
    const float* mp = a.m + x0 * NN;
    const float* mp0 = a.m + (x0 + 1 == N0 ? 0 : x0 + 1) * NN;
    const float* mm0 = a.m + (x0 == 0 ? N0 - 1 : x0 - 1) * NN;
    const int x2 = 16 * x2t + 4 * lk;
    const unsigned r = x1c * N2, rp = (x1c + 1 == N1 ? 0 : x1c + 1) * N2, rm = (x1c == 0 ? N1 - 1 : x1c - 1) * N2;
    o.c = row4(mp + r, x2, gs);
    o.lo = mp[r + (x2 == 0 ? N2 - 1 : min(x2, N2) - 1)];
    o.hi = mp[r + (x2 + 4 < N2 ? x2 + 4 : 0)];
    o.p0 = row4(mp0 + r, x2, gs);
    o.m0 = row4(mm0 + r, x2, gs);
    o.p1 = row4(mp + rp, x2, gs);
    o.m1 = row4(mp + rm, x2, gs);
    o.dm = a.dm ? row4(a.dm + x0 * NN + r, x2, gs) : make_float4(0.f, 0.f, 0.f, 0.f);
  };
  if constexpr (OP == GRID_SOURCE)
    if (wave < X2T) fetch(wave, near);

  for (int un = wave; un < 3 * KT; un += 4) {
    const int c = un % 3, kt = un / 3;
    // rows past Kh repeat the last one: they meet zero table entries
    const unsigned row = min(16 * kt + 4 * (li & 3) + (li >> 2), Kh - 1) * K1;
    const float2* plane = a.t1 + ((size_t)c * N0 + x0) * Kh * K1;
    floatx4 re, im;
    if constexpr (SEP) {
      floatx4 s0 = zero4(), s1 = zero4(), s2 = zero4(), s3 = zero4();
#pragma unroll 2
      for (int q = 0; q < KQ; ++q) {
        const float4 w0 = (f1 + ((size_t)x1t * 2 * KQ + q) * 64)[lane], w1 = (f1 + ((size_t)(x1t * 2 + 1) * KQ + q) * 64)[lane];
        float2 t[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) t[u] = plane[row + min(16 * q + 4 * u + lk, K1 - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const typename O::T tr = O::b(t[u].x), ti = O::b(t[u].y), wr = O::a(elem(w0, u)), wi = O::a(elem(w1, u));
          s0 = O::mma_t(tr, wr, s0);
          s1 = O::mma_t(ti, wi, s1);
          s2 = O::mma_t(ti, wr, s2);
          s3 = O::mma_t(tr, wi, s3);
        }
      }
      re = s0 - s1;
      im = s2 + s3;
    } else {
      re = im = zero4();
      for (int j0 = 0; j0 < J1; j0 += 4) {
        float4 w[4], t[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int j = min(j0 + q, J1 - 1);
          w[q] = (f1 + ((size_t)x1t * J1 + j) * 64)[lane];
          t[q] = ldu4(reinterpret_cast<const float*>(plane + (row + min(8 * j + 2 * lk, K1 - 2))));
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (j0 + q >= J1) break;
          float tr[4], ti[4];
          pair_operands(t[q], tr, ti);
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const float wi = elem(w[q], u), wr = flip(wi, neg);
            re = Op<false>::mma(tr[u], wr, re);
            im = Op<false>::mma(ti[u], wi, im);
          }
        }
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float* d = t2 + (c * 16 * KT + 16 * kt + 4 * r + lk) * S + li;
      d[0] = re[r];
      d[16] = im[r];
    }
  }
  __syncthreads();

  const size_t nN = (size_t)N0 * N1 * N2, plane0 = (size_t)x0 * N1 * N2;
  // table times stage-1 result: rows x2 and columns x1 for the source, rows x1
  // and columns x2 otherwise
  auto product = [&](float w, float t, floatx4 acc) {
    if constexpr (OP == GRID_SOURCE)
      return O::mma(O::a(w), O::b(t), acc);
    else
      return O::mma_t(O::b(t), O::a(w), acc);
  };
  float4 w[KT][2], wn[KT][2];
  auto table = [&](int x2t, float4 (&o)[KT][2]) {
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
      for (int q = 0; q < 2; ++q)
        if constexpr (SEP) o[kt][q] = (f2 + ((size_t)(x2t * 2 + q) * KT + kt) * 64)[lane];
        else o[kt][q] = (f2 + ((size_t)x2t * J2 + min(2 * kt + q, J2 - 1)) * 64)[lane];
  };
  table(min(wave, X2T - 1), w);
  for (int x2t = wave; x2t < X2T; x2t += 4) {
    table(min(x2t + 4, X2T - 1), wn);
    if constexpr (OP == GRID_SOURCE)
      if (x2t + 4 < X2T) fetch(x2t + 4, nxt);
    floatx4 vel[3];
    if constexpr (SEP) {
      floatx4 acc[3][2];
#pragma unroll
      for (int c = 0; c < 3; ++c) acc[c][0] = acc[c][1] = zero4();
#pragma unroll
      for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            const float* t = t2 + (c * 16 * KT + 16 * kt + 4 * u + lk) * S + li;
            acc[c][0] = product(elem(w[kt][0], u), t[0], acc[c][0]);
            acc[c][1] = product(elem(w[kt][1], u), t[16], acc[c][1]);
          }
#pragma unroll
      for (int c = 0; c < 3; ++c) vel[c] = acc[c][0] - acc[c][1];
    } else {
#pragma unroll
      for (int c = 0; c < 3; ++c) vel[c] = zero4();
#pragma unroll
      for (int j = 0; j < 2 * KT; ++j) {
        if (j >= J2) break;
        const float4 wj = w[j >> 1][j & 1];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int c = 0; c < 3; ++c)
            vel[c] = product(elem(wj, u), t2[(c * 16 * KT + 2 * (4 * j + u) + h) * S + part * 16 + li], vel[c]);
      }
    }
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
      for (int q = 0; q < 2; ++q) w[kt][q] = wn[kt][q];
    if constexpr (OP != GRID_SOURCE) {
      const int i2 = 16 * x2t + li;
      if (i2 >= N2) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i1 = 16 * x1t + 4 * lk + r;
        if (i1 >= N1) continue;
        const unsigned o = i1 * N2 + i2;
        if (OP == GRID_VELOCITY || a.vout) {
#pragma unroll
          for (int c = 0; c < 3; ++c) (a.vout + c * nN + plane0)[o] = vel[c][r];
        }
        if constexpr (OP == GRID_TRANSPORT)
          (a.dst + plane0)[o] =
              trilinear(a.src, (float)x0 - a.dt * vel[0][r] * (float)N0, (float)i1 - a.dt * vel[1][r] * (float)N1,
                        (float)i2 - a.dt * vel[2][r] * (float)N2, x0, i1, i2, gs);
      }
      continue;
    }
    const int x2 = 16 * x2t + 4 * lk;
    if (x1 < N1) {
      const float cc[6] = {near.lo, near.c.x, near.c.y, near.c.z, near.c.w, near.hi};
      const float p0[4] = {near.p0.x, near.p0.y, near.p0.z, near.p0.w}, m0[4] = {near.m0.x, near.m0.y, near.m0.z, near.m0.w};
      const float p1[4] = {near.p1.x, near.p1.y, near.p1.z, near.p1.w}, m1[4] = {near.m1.x, near.m1.y, near.m1.z, near.m1.w};
      const float dm[4] = {near.dm.x, near.dm.y, near.dm.z, near.dm.w};
      float q[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float up = (x2 + e + 1 < N2) ? cc[e + 2] : near.hi;  // the row's last point: its first
        const float g0 = (p0[e] - m0[e]) * (0.5f * N0);
        const float g1 = (p1[e] - m1[e]) * (0.5f * N1);
        const float g2 = (up - cc[e]) * (0.5f * N2);
        const float dot = g0 * vel[0][e] + g1 * vel[1][e] + g2 * vel[2][e];
        q[e] = fmaf(-a.dt, dot, dm[e]);
      }
      put4(a.q + plane0 + (size_t)x1 * N2, x2, make_float4(q[0], q[1], q[2], q[3]), gs);
    }
    near = nxt;
  }
}

hipError_t launch_gridstep_chain(const GridStepArgs& a, const Dims& d, const Frags& fr, hipStream_t st) {
  if (grid_instantiated(d) ? (!fr.row1 || !fr.row2) : (!fr.inv1 || !fr.inv2)) return hipErrorInvalidValue;
  const dim3 grid(tiles16(d.N[1]), d.N[0]);
  return with_grid(d, [&](auto gs) -> hipError_t {
    using G = decltype(gs);
    if constexpr (G::kStatic) {
      if (a.op != GRID_TRANSPORT) return hipErrorInvalidValue;
      if (d.prec)
        LAUNCH_TIMED(KF_GRID, (k_gridstep<1, GRID_TRANSPORT, true, true, G>), grid, dim3(256), 0, st, a, fr.row1, fr.row2, gs);
      else
        LAUNCH_TIMED(KF_GRID, (k_gridstep<1, GRID_TRANSPORT, true, false, G>), grid, dim3(256), 0, st, a, fr.row1, fr.row2, gs);
      return hipGetLastError();
    } else {
      return with_int<2>(tiles16(d.Kh), [&](auto kt) {
        constexpr int KT = decltype(kt)::value;
        if (a.op == GRID_VELOCITY)
          LAUNCH_TIMED(KF_GRID, (k_gridstep<KT, GRID_VELOCITY, false, false, G>), grid, dim3(256), 0, st, a, fr.inv1, fr.inv2, gs);
        else if (a.op == GRID_SOURCE)
          LAUNCH_TIMED(KF_GRID, (k_gridstep<KT, GRID_SOURCE, false, false, G>), grid, dim3(256), 0, st, a, fr.inv1, fr.inv2, gs);
        else
          LAUNCH_TIMED(KF_GRID, (k_gridstep<KT, GRID_TRANSPORT, false, false, G>), grid, dim3(256), 0, st, a, fr.inv1, fr.inv2, gs);
        return hipGetLastError();
      });
    }
  });
}

}  // namespace lddmm
