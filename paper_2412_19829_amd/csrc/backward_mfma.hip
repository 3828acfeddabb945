// Backward pass of the windowed softmax heads on bf16 matrix cores (section III-B, Eq. 1,
// differentiated; the formulas are stated at the top of backward_scalar.hip).
//
// With s_ij = scale q_i.k_j, p_ij the softmax over the causal window, dp_ij = dO_i.v_j,
// D_i = sum_j p_ij dp_ij and ds_ij = p_ij (dp_ij - D_i):
//   dq_i = scale sum_j ds_ij k_j,   dk_j = scale sum_i ds_ij q_i,   dv_j = sum_i p_ij dO_i.
//
// Every one of these is a band product like the forward pass: 32 "resident" rows per wave (their
// operands stay in registers) against the band of "streamed" rows they interact with, walked in
// tiles of 64 rows that pass through LDS.  One template, four passes:
//   kStats  resident queries (q, dO), streamed keys (K, V): log-sum-exp and D_i of every query,
//           left in the workspace;
//   kDq     the same band again: ds from the stored statistics, dq^T += K^T ds^T;
//   kDv     resident keys (k), streamed queries (Q, dO): dv^T += dO^T p;
//   kDk     resident keys (k, v), streamed queries (Q, dO): dk^T += Q^T ds.
// Scores are computed with the streamed rows as MFMA rows and the resident rows as columns, so a
// lane owns one resident row; the weights then feed the output product straight from the score
// registers (the k-index permutation of an accumulator tile used as an operand is matched by the
// order in which the transposed LDS read delivers the streamed tile).
//
// Arithmetic: bf16 products with fp32 accumulation; the softmax statistics, D_i and ds in fp32;
// p and ds are rounded to bf16 as operands of the output product.  Nothing of the forward result
// is an input.
#include "backward_band.hpp"

namespace gformer {
namespace {

template <int D, int PASS>
__global__ __launch_bounds__(kBandThreads, 2) void windowed_bwd_band_kernel(BwdArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  windowed_band<D, PASS>(a, blockIdx.x, smem_raw);
}

template <int D> hipError_t launch_windowed_bwd_t(const BwdArgs& a, bool statistics_only, hipStream_t s) {
  constexpr int BR = band_rows(kBandThreads);
  const dim3 grid(((a.N + BR - 1) / BR) * a.H0 * a.B), block(kBandThreads);
  const int smem = (int)sizeof(BandSmem<D>);
  hipError_t e = hipSuccess;
  auto launch = [&](auto kern) {
    if (e != hipSuccess) return;
    e = allow_lds(kern, smem);
    if (e == hipSuccess) kern<<<grid, block, smem, s>>>(a);
  };
  launch(windowed_bwd_band_kernel<D, kStats>);
  if (statistics_only) return e != hipSuccess ? e : hipGetLastError();
  launch(windowed_bwd_band_kernel<D, kDq>);
  launch(windowed_bwd_band_kernel<D, kDv>);
  launch(windowed_bwd_band_kernel<D, kDk>);
  return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace

// Windowed heads [0, H0) of a bf16 call; the workspace receives (log2-sum-exp, D_i) per query.
hipError_t launch_windowed_backward_mfma(const BwdArgs& a, hipStream_t s, bool statistics_only) {
  if (a.H0 <= 0 || a.N <= 0 || a.B <= 0) return hipSuccess;
  return a.d == 64 ? launch_windowed_bwd_t<64>(a, statistics_only, s) : launch_windowed_bwd_t<128>(a, statistics_only, s);
}

}  // namespace gformer
