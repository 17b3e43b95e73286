// Synthesis and Lie products of a step in one launch (small bands).
#include <algorithm>

#include "launch.h"
#include "lie.h"
#include "mfma.h"
#include "shapes.h"

namespace lddmm {
namespace {

// New fields, products and cached groups of a program (ProdArgs::g holds the
// new groups first).
constexpr int step_fields(int prog) { return prog == PROG_ADJ || prog == PROG_DEF_FWD || prog == PROG_DEF_H ? 3 : 6; }
constexpr int step_outs(int prog) {
  return prog == PROG_GRAD || prog == PROG_H5 ? 9 : prog == PROG_ADJ ? 6 : 3;
}
constexpr int step_cached(int prog) {
  return prog == PROG_SHOOT ? 0 : prog == PROG_H5 ? 6 : prog == PROG_DEF_FWD ? 1 : prog == PROG_DEF_H ? 3 : 2;
}

// One block per (x0 plane, 16 x1): inverse stages 1 and 2 of the step's new
// fields, the products of the program with them and the cached groups, and
// the products' forward stage 2, in the orders of k_synth_chain and k_prods.
//   1  wave (field, stage-0 input): stage 1 (k1 -> x1) against the plain and the
//      derivative table, or the plain one; T2 goes to LDS as the operand of
//   2  wave (x2 tile, field, half): stage 2 (k2 -> x2), two of a point's four
//      values (value and d2, or d0 and d1), to LDS
//   3  thread (point): the new groups leave (where the caller keeps them), the
//      products meet in the LDS of T2
//   4  wave (product): forward stage 2 (x2 -> kh).
// The cached groups are read at the start, into registers, and arrive during
// phases 1 and 2.  Every load is of consecutive addresses: one whose 16-lane
// quarters touch 16 rows each keeps the address unit for 64 cycles.  Bound by the chain of latencies (its products take 4 us of the
// matrix cores of 144 compute units at band 32): what it saves against a
// synthesis and a product launch is the second launch, its load phase and the
// fields' way through memory.
// Band 32 (M = 48), alone: 21 us (9 + 12) as two launches, 13 to 15 so; band 8
// (M = 12): 5.6 + 4.5 us as two, 6.2 so.
template <int PROG, int KQ, bool BF3>
__global__ void __launch_bounds__(768) k_step(StepArgs a, const float4* __restrict__ fr1,
                                              const float4* __restrict__ fr2, const float2* __restrict__ fwd2,
                                              BandDyn sh) {
  using O = Op<BF3>;
  constexpr int NF = step_fields(PROG), NOUT = step_outs(PROG), NC = step_cached(PROG);
  extern __shared__ float lds[];
  const int M0 = sh.M0(), M1 = sh.M1(), M2 = sh.M2(), K1 = sh.K1(), Kh = sh.Kh();
  const int X1T = (M1 + 15) / 16, X2T = (M2 + 15) / 16;
  const int L4 = (M2 + 3) & ~3, LV = 4 * ((L4 / 4) | 1), LF = 16 * X2T + 4;
  float4* t2s = reinterpret_cast<float4*>(lds);  // [NF][value, d1, d0][re, im][64]
  float* vals = lds;                             // [NOUT][16][LV], in its place
  float2* fs = reinterpret_cast<float2*>(lds + max(NF * 6 * 64 * 4, NOUT * 16 * LV));  // [NF][2][16][LF]
  float2* ts = fs;                                                          // [NF][2][Kh][LT], in its place
  const int LT = row_ld(K1), LW = row_ld(M2);
  float2* ws = fs + NF * 2 * 16 * max(LF, LT);                              // [Kh][LW]
  const int wave = wave_id(), lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int waves = blockDim.x >> 6;
  const int x0 = blockIdx.y, x1t = blockIdx.x;

  // What phases 1 and 2 read; the cached groups follow when phase 1's input is
  // there (loads return in the order of their issue: no phase waits for a later
  // one's, and no wave for another's).
  const int f1 = wave % NF, vs1 = wave / NF;
  constexpr int NT = 2 * KQ;  // 1 KB loads of a stage-0 input [Kh][K1]
  floatx4 tr[NT];
  float4 w[2][2 * KQ];
  const int npair = Kh * K1 / 2;
  if (wave < 2 * NF) {
    const floatx4* plane =
        reinterpret_cast<const floatx4*>(a.t1[f1 / 3] + (unsigned)((((f1 % 3) * 2 + vs1) * M0 + x0) * Kh * K1));
#pragma unroll
    for (int i = 0; i < NT; ++i) tr[i] = plane[min(64 * i + lane, npair - 1)];
#pragma unroll
    for (int pq = 0; pq < 2 * KQ; ++pq) w[0][pq] = (fr1 + (x1t * 2 * KQ + pq) * 64)[lane];
    if (!vs1) {
#pragma unroll
      for (int pq = 0; pq < 2 * KQ; ++pq) w[1][pq] = (fr1 + ((X1T + x1t) * 2 * KQ + pq) * 64)[lane];
    }
  }
  // phase 2: this wave's (x2 tile, half), and which of the fields
  const int half = wave & 1, x2t = (wave >> 1) % X2T, f2 = wave / (2 * X2T), f2n = waves / (2 * X2T);
  float4 w0[2], w1[2];
#pragma unroll
  for (int part = 0; part < 2; ++part) {
    w0[part] = (fr2 + (2 * x2t + part) * 64)[lane];
    w1[part] = (fr2 + ((half ? 0 : 2 * X2T) + 2 * x2t + part) * 64)[lane];
  }
  const float2 wt = fwd2[min((int)threadIdx.x, Kh * M2 - 1)];
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  // this thread's point and its cached values (value, d0, d1, d2 per component);
  // of six groups two wait until stage 1 has freed its registers
  const int pr = threadIdx.x / L4, px = threadIdx.x - pr * L4, px1 = 16 * x1t + pr;
  const bool valid = pr < 16 && px1 < M1 && px < M2;
  const unsigned nM = (unsigned)(M0 * M1 * M2);
  const unsigned gp = (unsigned)((x0 * M1 + min(px1, M1 - 1)) * M2 + min(px, M2 - 1));
  constexpr int NE = NC > 4 ? 4 : NC;
  float4 c[NC > 0 ? NC : 1][3];
  auto cached = [&](int k) {
#pragma unroll
    for (int i = 0; i < 3; ++i) c[k][i] = reinterpret_cast<const float4*>(a.cached[k])[i * nM + gp];
  };
  // 1: stage 1, this wave's input turned in LDS
  if (wave < 2 * NF) {
    float2* tl = ts + (f1 * 2 + vs1) * 16 * LT;
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int at = 2 * (64 * i + lane), kh = at / K1;
      if (64 * i + lane < npair) *reinterpret_cast<floatx4*>(tl + kh * LT + (at - kh * K1)) = tr[i];
    }
    // (their loads would be ahead of other waves' inputs before this point)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < NE; ++k) cached(k);
    __builtin_amdgcn_sched_barrier(0);
    float2 t[KQ][4];
    {
      // rows past Kh and k1 past K1 repeat the last one: they meet zero table entries
      const float2* row = tl + min(4 * (li & 3) + (li >> 2), Kh - 1) * LT;
#pragma unroll
      for (int q = 0; q < KQ; ++q)
#pragma unroll
        for (int u = 0; u < 4; ++u) t[q][u] = row[min(16 * q + 4 * u + lk, K1 - 1)];
    }
    auto stage1 = [&](auto VS) {
      constexpr int vs = decltype(VS)::value, NV = vs ? 1 : 2;
      floatx4 acc[NV][2];
#pragma unroll
      for (int v = 0; v < NV; ++v) acc[v][0] = acc[v][1] = zero4();
#pragma unroll
      for (int pq = 0; pq < 2 * KQ; ++pq) {
        const int part = pq / KQ, q = pq % KQ;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float tx = t[q][u].x, ty = t[q][u].y;
          const typename O::T yr = O::b(part ? ty : tx), yi = O::b(part ? -tx : ty);
#pragma unroll
          for (int v = 0; v < NV; ++v) {
            const typename O::T x = O::a(elem(w[v][pq], u));
            acc[v][0] = O::mma_t(yr, x, acc[v][0]);
            acc[v][1] = O::mma_t(yi, x, acc[v][1]);
          }
        }
      }
#pragma unroll
      for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int q = 0; q < 2; ++q)
          t2s[((f1 * 3 + (vs ? 2 : v)) * 2 + q) * 64 + lane] =
              make_float4(acc[v][q][0], acc[v][q][1], acc[v][q][2], acc[v][q][3]);
    };
    if (vs1)
      stage1(std::integral_constant<int, 1>{});
    else
      stage1(std::integral_constant<int, 0>{});
  } else {
#pragma unroll
    for (int k = 0; k < NE; ++k) cached(k);
  }
#pragma unroll
  for (int k = NE; k < NC; ++k) cached(k);
  __syncthreads();

  // 2: stage 2
  for (int f = f2; f2 < f2n && f < NF; f += f2n) {
    floatx4 g0 = zero4(), g1 = zero4();
    float4 p0[2], p1[2];
#pragma unroll
    for (int part = 0; part < 2; ++part) {
      p0[part] = t2s[((f * 3 + (half ? 2 : 0)) * 2 + part) * 64 + lane];
      p1[part] = t2s[((f * 3 + (half ? 1 : 0)) * 2 + part) * 64 + lane];
    }
#pragma unroll
    for (int part = 0; part < 2; ++part)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        g0 = O::mma(O::a(elem(p0[part], u)), O::b(elem(w0[part], u)), g0);
        g1 = O::mma(O::a(elem(p1[part], u)), O::b(elem(w1[part], u)), g1);
      }
    float2* out = fs + ((f * 2 + half) * 16 + 4 * lk) * LF + 16 * x2t + li;
#pragma unroll
    for (int r = 0; r < 4; ++r) out[r * LF] = make_float2(g0[r], g1[r]);
  }
  if ((int)threadIdx.x < Kh * M2) ws[(threadIdx.x / M2) * LW + threadIdx.x % M2] = wt;
  __syncthreads();

  // 3: products
  if (pr < 16) {
    float g[NF / 3][12];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const float2 e = fs[((f * 2) * 16 + pr) * LF + px], d = fs[((f * 2 + 1) * 16 + pr) * LF + px];
      float* q = g[f / 3];
      q[f % 3] = e.x;
      q[3 + 3 * (f % 3)] = d.x;
      q[4 + 3 * (f % 3)] = d.y;
      q[5 + 3 * (f % 3)] = e.y;
      if (a.dst[f / 3] && valid)
        reinterpret_cast<float4*>(a.dst[f / 3])[(f % 3) * nM + gp] = make_float4(e.x, d.x, d.y, e.y);
    }
    float h[NC > 0 ? NC : 1][12];
#pragma unroll
    for (int k = 0; k < NC; ++k)
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        h[k][i] = c[k][i].x;
        h[k][3 + 3 * i] = c[k][i].y;
        h[k][4 + 3 * i] = c[k][i].z;
        h[k][5 + 3 * i] = c[k][i].w;
      }
    float o[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) o[i] = 0.f;
    if constexpr (PROG == PROG_SHOOT) {  // new: V, LV
      adstar_acc(o, g[0], g[1], 1.f);
    } else if constexpr (PROG == PROG_H1) {  // new: dV, LdV; cached: V, LV
      adstar_acc(o, g[0], h[1], 1.f);
      adstar_acc(o, h[0], g[1], 1.f);
    } else if constexpr (PROG == PROG_GRAD) {  // new: LU, W (or LdU, dW); cached: V, LV
      adstar_acc(o, h[0], g[0], 1.f);
      ad_acc(o + 3, h[0], g[1], 1.f);
      adstar_acc(o + 6, g[1], h[1], 1.f);
    } else if constexpr (PROG == PROG_H5) {  // new: LdU, dW; cached: V, LV, LU, W, dV, LdV
      adstar_acc(o, h[0], g[0], 1.f);
      ad_acc(o + 3, h[0], g[1], 1.f);
      adstar_acc(o + 6, g[1], h[1], 1.f);
      adstar_acc(o, h[4], h[2], 1.f);
      ad_acc(o + 3, h[4], h[3], 1.f);
      adstar_acc(o + 6, h[3], h[5], 1.f);
    } else if constexpr (PROG == PROG_ADJ) {  // new: W; cached: V, LV
      ad_acc(o, h[0], g[0], 1.f);
      adstar_acc(o + 3, g[0], h[1], 1.f);
    } else if constexpr (PROG == PROG_DEF_FWD) {  // new: Phi; cached: V
      jac_acc(o, g[0] + 3, h[0]);
    } else {  // PROG_DEF_H, new: dPhi; cached: V, Phi, dV
      jac_acc(o, g[0] + 3, h[0]);
      jac_acc(o, h[1] + 3, h[2]);
    }
#pragma unroll
    for (int i = 0; i < NOUT; ++i) vals[(i * 16 + pr) * LV + px] = valid ? o[i] : 0.f;
  }
  __syncthreads();

  // 4: forward stage 2
  for (int o = wave; o < NOUT; o += waves) {
    const float* row = vals + (o * 16 + li) * LV + lk;
    const float2* wr = ws + min(li, Kh - 1) * LW;
    constexpr int KS = kStepM2 / 4;
    float v[KS];
    float2 wf[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      v[ks] = row[min(4 * ks, L4 - 4)];
      wf[ks] = wr[min(4 * ks + lk, M2 - 1)];
    }
    floatx4 re = zero4(), im = zero4();
    auto sum = [&](auto B) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        if (4 * ks >= M2) break;
        using P = Op<decltype(B)::value>;
        const typename P::T x = P::a(v[ks]);
        re = P::mma_t(P::b(wf[ks].x), x, re);
        im = P::mma_t(P::b(wf[ks].y), x, im);
      }
    };
    // rows that are no whole k-steps are summed in FP32 in either precision
    if (BF3 && M2 % 4 == 0)
      sum(std::integral_constant<bool, true>{});
    else
      sum(std::integral_constant<bool, false>{});
    // rows kh, columns x1: 128-byte runs
    const int x1 = 16 * x1t + li;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int kh = 4 * lk + r;
      if (x1 < M1 && kh < Kh) a.s1[(unsigned)(((o * Kh + kh) * M0 + x0) * M1 + x1)] = make_float2(re[r], im[r]);
    }
  }
}

// LDS of a block: T2 or the products, the fields, the table of forward stage 2.
constexpr size_t step_bytes(int nf, int nout, int K1, int Kh, int M2) {
  const int L4 = (M2 + 3) & ~3, LV = 4 * ((L4 / 4) | 1), LF = 16 * tiles16(M2) + 4;
  return ((size_t)std::max(nf * 6 * 64 * 4, nout * 16 * LV) + 2 * (size_t)nf * 2 * 16 * std::max(LF, row_ld(K1)) +
          2 * (size_t)Kh * row_ld(M2)) * sizeof(float);
}

template <int PROG>
hipError_t launch_prog(const StepArgs& a, const Frags& fr, const float2* fwd2, const Dims& d, hipStream_t st) {
  constexpr int NF = step_fields(PROG), NOUT = step_outs(PROG);
  for (int k = 0; k < step_cached(PROG); ++k)
    if (!a.cached[k]) return hipErrorInvalidValue;
  if (!a.t1[0] || (NF == 6 && !a.t1[1]) || !a.s1) return hipErrorInvalidValue;
  const BandDyn sh{d.K[0], d.K[1], d.Kh, d.M[0], d.M[1], d.M[2]};
  const size_t shm = step_bytes(NF, NOUT, d.K[1], d.Kh, d.M[2]);
  static_assert(step_bytes(NF, NOUT, 32, 16, kStepM2) <= kMaxLds);
  const int L4 = (d.M[2] + 3) & ~3;
  const dim3 grid(tiles16(d.M[1]), d.M[0]), block(64 * std::max(2 * NF, (16 * L4 + 63) / 64));
  auto go = [&](auto kq, auto bf) {
    constexpr int KQ = decltype(kq)::value;
    constexpr bool B = decltype(bf)::value;
    LAUNCH_TIMED(KF_PRODS, (k_step<PROG, KQ, B>), grid, block, shm, st, a, fr.row1, fr.row2, fwd2, sh);
    return hipGetLastError();
  };
  auto by_prec = [&](auto kq) {
    return d.prec ? go(kq, std::integral_constant<bool, true>{}) : go(kq, std::integral_constant<bool, false>{});
  };
  return d.K[1] <= 16 ? by_prec(std::integral_constant<int, 1>{}) : by_prec(std::integral_constant<int, 2>{});
}
}  // namespace

// One tile of kh, two of k1 and three of x2: what a block's LDS (123 KB of 160) and
// a wave's registers hold.  Past it the fields of a block do not fit and two
// launches are the only form; inside it one launch was faster at every band
// tried (8, 16, 24, 32).
bool step_fused(const Dims& d) { return d.Kh <= 16 && d.K[1] <= 32 && d.M[2] <= kStepM2; }

hipError_t launch_step(int prog, const StepArgs& a, const Frags& fr, const Twiddles& tw, const Dims& d,
                       hipStream_t st) {
  if (!step_fused(d) || !fr.row1 || !fr.row2 || !tw.fwd2) return hipErrorInvalidValue;
  {
    const double nM = (double)d.nM;
    static const double flops[11] = {0, 47, 94, 136, 272, 136, 18, 36, 18, 36, 89};
    const int p = prog == PROG_H5_NOCOUPLE ? PROG_GRAD : prog;
    const int nf = step_fields(p), no = step_outs(p);
    const int kept = (a.dst[0] ? 3 : 0) + (a.dst[1] ? 3 : 0);
    timer_work(KF_PRODS,
               nf * (3.0 * d.M[0] * d.M[1] * d.Kh * d.K[1] * 8.0 + 4.0 * nM * d.Kh * 4.0) + flops[prog] * nM +
                   no * nM * d.Kh * 4.0,
               nf * 2.0 * d.M[0] * d.K[1] * d.Kh * 8.0 + (kept + 3.0 * step_cached(p)) * nM * 16.0 +
                   no * (double)d.M[0] * d.M[1] * d.Kh * 8.0);
  }
  switch (prog) {
    case PROG_SHOOT: return launch_prog<PROG_SHOOT>(a, fr, tw.fwd2, d, st);
    case PROG_H1: return launch_prog<PROG_H1>(a, fr, tw.fwd2, d, st);
    case PROG_GRAD:
    case PROG_H5_NOCOUPLE: return launch_prog<PROG_GRAD>(a, fr, tw.fwd2, d, st);
    case PROG_H5: return launch_prog<PROG_H5>(a, fr, tw.fwd2, d, st);
    case PROG_ADJ: return launch_prog<PROG_ADJ>(a, fr, tw.fwd2, d, st);
    case PROG_DEF_FWD: return launch_prog<PROG_DEF_FWD>(a, fr, tw.fwd2, d, st);
    case PROG_DEF_H: return launch_prog<PROG_DEF_H>(a, fr, tw.fwd2, d, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace lddmm
