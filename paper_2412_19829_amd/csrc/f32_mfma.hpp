// Helpers of the single-precision matrix-core kernels (v_mfma_f32_16x16x4_f32: fp32 operands, fp32
// accumulation, 256 FLOP per cycle and compute unit, twice what plain FMAs give).
//
// Lane layout (D = A*B + C, A is 16x4, B is 4x16), lane l, g = l/16:
//   A operand: row m = l%16, k-slot g      B operand: column n = l%16, k-slot g
//   C/D:       column n = l%16, register r holds row m = 4*g + r
// The four k-slots of an instruction may stand for any four indices as long as A and B agree, so
//   - a contraction along the rows of two LDS tiles takes 16 consecutive columns per four
//     instructions: lane l reads columns 16*kk + 4*g .. +3 of its row with one 16-byte load, and
//     instruction j uses element j of both (rows_product);
//   - an accumulator tile feeds the next product straight from its registers: register r is the
//     operand of the instruction whose k-slots are rows r, 4 + r, 8 + r, 12 + r;
//   - where the output's row index runs along a tile's columns, tile x of a group of four takes
//     columns 4*i + x, i = 0..15, so one 16-byte load per lane serves four instructions and a
//     lane ends up with four consecutive columns (64*hh + 16*g + 4*r + x, x = 0..3).
// LDS rows are D + 4 floats apart: 16-byte aligned, and rows 4 apart start 16 banks apart.
#pragma once

#include "common.hpp"

namespace gformer {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 lds4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
constexpr f32x4 kZeroF4 = {0.f, 0.f, 0.f, 0.f};

template <int D> constexpr int kF32Row = D + 4;   // LDS row stride in floats

// Sum / maximum over the four lanes l%16 + 16*g; every lane gets the result.
__device__ __forceinline__ float sum_over_groups(float x) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float max_over_groups(float x) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// 16x16 tile of products of rows: result row m = row m of `a_rows`, column n = row n of the operand
// held in registers (element 4*kk + j = column 16*kk + 4*g + j).  Two accumulators taken in turn.
template <int D>
__device__ __forceinline__ f32x4 rows_product(const float* a_lane, const float (&b)[D / 4]) {
  f32x4 acc0 = kZeroF4, acc1 = kZeroF4;
#pragma unroll
  for (int kk = 0; kk < D / 16; kk += 2) {
    const f32x4 x = lds4(a_lane + 16 * kk), y = lds4(a_lane + 16 * kk + 16);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      acc0 = mfma_f32(x[j], b[4 * kk + j], acc0);
      acc1 = mfma_f32(y[j], b[4 * kk + 4 + j], acc1);
    }
  }
  return acc0 + acc1;
}
// The same with both operands in LDS.
template <int D>
__device__ __forceinline__ f32x4 rows_product_lds(const float* a_lane, const float* b_lane) {
  f32x4 acc0 = kZeroF4, acc1 = kZeroF4;
#pragma unroll
  for (int kk = 0; kk < D / 16; kk += 2) {
    const f32x4 x = lds4(a_lane + 16 * kk), y = lds4(a_lane + 16 * kk + 16);
    const f32x4 u = lds4(b_lane + 16 * kk), w = lds4(b_lane + 16 * kk + 16);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      acc0 = mfma_f32(x[j], u[j], acc0);
      acc1 = mfma_f32(y[j], w[j], acc1);
    }
  }
  return acc0 + acc1;
}

}  // namespace
}  // namespace gformer
