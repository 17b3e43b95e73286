// Matrix-core operands and the fragment tables of the chained partial DFTs.
#pragma once

#include "common.h"

namespace lddmm {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// Compensated BF16 products on the matrix cores (precision LDDMM_FP32_BF16X3):
// each FP32 operand x is split as hi = bf16(x), lo = bf16(x - hi) (round to
// nearest even both times), and a b is formed as ah bh + ah bl + al bh with
// FP32 accumulation; the dropped al bl is about 2^-16 of a b.  One FP32
// k-step of v_mfma_f32_16x16x4f32 becomes one v_mfma_f32_16x16x16_bf16 whose
// four k slots per lane hold the three terms and a zero: the A operand
// (ah, ah, al, 0), the B operand (bh, bl, bh, 0).  Both operands index k
// by (lane / 16, slot) alike, so the slot order only has to pair the terms.
__device__ __forceinline__ shortx4 bf3_a(float x) {
  const __bf16 h = (__bf16)x;
  const __bf16 l = (__bf16)(x - (float)h);
  const bf16x4 v = {h, h, l, (__bf16)0.f};
  return __builtin_bit_cast(shortx4, v);
}
__device__ __forceinline__ shortx4 bf3_b(float x) {
  const __bf16 h = (__bf16)x;
  const __bf16 l = (__bf16)(x - (float)h);
  const bf16x4 v = {h, l, h, (__bf16)0.f};
  return __builtin_bit_cast(shortx4, v);
}
__device__ __forceinline__ floatx4 mma_bf3(shortx4 a, shortx4 b, floatx4 acc) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, acc, 0, 0, 0);
}
// acc += a b over one k-step of a 16x16 tile (lane layout of
// v_mfma_f32_16x16x4f32: A[row = lane % 16][k = lane / 16], B[k][col = lane % 16]).
template <bool BF3>
__device__ __forceinline__ floatx4 mma(float a, float b, floatx4 acc) {
  if constexpr (BF3)
    return mma_bf3(bf3_a(a), bf3_b(b), acc);
  else
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc, 0, 0, 0);
}

// An operand split once and used in several products.
template <bool BF3>
struct Op;
template <>
struct Op<false> {
  using T = float;
  static __device__ __forceinline__ float a(float x) { return x; }
  static __device__ __forceinline__ float b(float x) { return x; }
  static __device__ __forceinline__ floatx4 mma(float x, float y, floatx4 acc) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(x, y, acc, 0, 0, 0);
  }
  // the B form as the first operand: the transposed tile
  static __device__ __forceinline__ floatx4 mma_t(float y, float x, floatx4 acc) { return mma(y, x, acc); }
};
template <>
struct Op<true> {
  using T = shortx4;
  static __device__ __forceinline__ shortx4 a(float x) { return bf3_a(x); }
  static __device__ __forceinline__ shortx4 b(float x) { return bf3_b(x); }
  static __device__ __forceinline__ floatx4 mma(shortx4 x, shortx4 y, floatx4 acc) { return mma_bf3(x, y, acc); }
  static __device__ __forceinline__ floatx4 mma_t(shortx4 y, shortx4 x, floatx4 acc) { return mma_bf3(y, x, acc); }
};

// Index of this wave in its block, as a value the compiler knows to be the same
// in all lanes (addresses built from it stay in scalar registers).
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

// Row stride of complex values read 16 rows at a time: twice an odd number.
__host__ __device__ constexpr int row_ld(int n) { return 2 * (((n + 1) / 2) | 1); }

__device__ __forceinline__ floatx4 zero4() { return floatx4{0.f, 0.f, 0.f, 0.f}; }

// ------------------------------------------------------------ chained stages
// A transform of the shapes without instantiated kernels is a chain of matrix
// products whose operands come straight from memory and whose tables are
// kept in the order in which a wave reads them (1 KB rows of 64 lanes).
// Two facts carry it.
//   * The result of a 16x16 tile holds, in lane (li = lane % 16, lk = lane /
//     16) and register r, element (row 4 lk + r, column li); as the A operand
//     (row li) or the B operand (column li) of a next product, register u is
//     what lane lk has to supply for k-step u.  Which row of the product is
//     called 4 lk + r is free, so a stage names its rows in the order in
//     which the next stage counts them.
//   * v_mfma_f32_16x16x4f32 adds its four products one after the other, each
//     a fused multiply-add: a chain of them is the sequential sum over k,
//     whichever operand is called A, and zero entries change nothing.  So the
//     sums below are formed in the order in which scalar code would form them
//     (and the energies, which are returned in double, do not depend on which
//     kernel a shape runs on).
// Orders of a complex sum  sum_k w(k) t(k):
//   rows   all k with re w, then all k with -im w: k-step u of group q of a part
//          holds k = 16 q + 4 u + lk;
//   pairs  per k first re w, then -im w (for the imaginary part im w): k-step
//          ks holds k = 2 ks + lk / 2, part lk % 2.
// Fragment tables (k_tables), row or column index 16 tile + li, zero padded:
//   ROW_INV   [v][x tile][part][k tile][64] float4: re w (part 0) or -im w of
//             u = 0 .. 3; v = 1: w times 2 pi i k; the half form runs over
//             k = 0 .. Kh - 1 with weight 1 at k = 0, else 2
//   ROW_INV_POS  the same with im w in part 1, for kernels that form the parts
//             apart and subtract: v_mfma_f32_16x16x16_bf16 does not round x and -x
//             alike, so the sign a table holds decides the last bits of the
//             compensated products (FP32 sums are the same either way)
//   PAIR_INV  [v][x tile][ks / 4][64] float4: this lane's part of w (re or im)
//             for four k-steps; the half form (real output) holds re and -im
//   PAIR_FWD  [k tile][ks / 4][64] float4: the same with x = 2 ks + lk / 2
__device__ __forceinline__ float elem(const float4& v, int s) {
  return s == 0 ? v.x : s == 1 ? v.y : s == 2 ? v.z : v.w;
}
__device__ __forceinline__ float flip(float x, unsigned sign) {
  return __uint_as_float(__float_as_uint(x) ^ sign);
}

// Rows of 16 lanes lk = 0 .. 3 hold (x, y) = values 2 lk and 2 lk + 1 of eight:
// after the exchange x holds value lk, y value 4 + lk (two k-steps of four from
// one load of consecutive values).
__device__ __forceinline__ void swap_quarters(float& x, float& y) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(a[0], a[1], false, false);
  x = __uint_as_float(b[0]);
  y = __uint_as_float(b[1]);
}

// A lane of row lk holds complex elements 2 lk (v.x, v.y) and 2 lk + 1 (v.z,
// v.w) of eight: the operands of four k-steps in "pairs" order, k-step s element
// 2 s + lk / 2, the part of it that meets re w (lk even) or im w (lk odd).
__device__ __forceinline__ void pair_operands(const float4& v, float (&re)[4], float (&im)[4]) {
  auto four = [](float x0, float y0, float x1, float y1, float (&o)[4]) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x0), __float_as_uint(y0), false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x1), __float_as_uint(y1), false, false);
    const auto e = __builtin_amdgcn_permlane32_swap(a[0], b[0], false, false);
    const auto f = __builtin_amdgcn_permlane32_swap(a[1], b[1], false, false);
    o[0] = __uint_as_float(e[0]);
    o[1] = __uint_as_float(f[0]);
    o[2] = __uint_as_float(e[1]);
    o[3] = __uint_as_float(f[1]);
  };
  four(v.x, v.y, v.z, v.w, re);
  four(v.y, v.x, v.w, v.z, im);
}

// 16-byte loads and stores of 4- or 8-byte aligned addresses
typedef float f4_u4 __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ float4 ldu4(const float* p) {
  const f4_u4 v = *reinterpret_cast<const f4_u4*>(p);
  return make_float4(v.x, v.y, v.z, v.w);
}

// Logical block index (x, y, z) of a launch whose workgroups the command
// processor hands round-robin to the eight XCDs (workgroup p to XCD p % 8):
// with the block count a multiple of 8, XCD x takes the contiguous logical
// range [x T/8, (x + 1) T/8), so blocks that are neighbours in the logical
// order run on one XCD and meet in its L2.  The logical order runs x fastest,
// or with ZFirst z fastest, then x, then y (for launches whose z blocks of
// one (x, y) read the same input: the column steps' k1 tiles and parts of one
// kh read the same stage-1 input, and neighbouring kh share 32-byte granules
// of the band).
template <bool ZFirst>
__device__ __forceinline__ uint3 xcd_block3() {
  const unsigned gx = gridDim.x, gy = gridDim.y, gz = gridDim.z, total = gx * gy * gz;
  unsigned p = blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z);
  if (total % 8u == 0) p = (p % 8u) * (total / 8u) + p / 8u;
  if constexpr (ZFirst) return make_uint3((p / gz) % gx, p / (gz * gx), p % gz);
  return make_uint3(p % gx, (p / gx) % gy, p / (gx * gy));
}

}  // namespace lddmm
