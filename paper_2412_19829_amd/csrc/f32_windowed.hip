// Windowed softmax heads in single precision on the matrix cores: forward (section III-B, Eq. 1)
// and backward (its derivatives, see backward_scalar.hip), causal or centred windows.
//
// The work is products of 16 resident rows with the rows of a band: 16x16 tiles of scores, whose
// registers are the weights' operand of the product that follows (f32_mfma.hpp), so weights never
// leave a wave.  The band is walked in tiles of 64 rows staged in LDS for the four waves of a
// workgroup.  QB of the waves hold 16 resident rows each and the other 4 / QB share them, taking
// every (4 / QB)-th group of 16 band rows: QB = 4 reads every tile once per 64 rows, QB = 1 makes
// four times as many workgroups and is taken while 64-row workgroups would leave compute units idle.
//
// Measured, 12 heads, N=2048, d=64, w=128 (plain-FMA kernels -> these, us): forward 319 -> 24, dq 296 -> 48,
// dk and dv 403 -> 37.  Bound: the SIMDs' issue; the matrix core is busy 27-33 % of the time, and 384
// workgroups of 64 rows leave every other compute unit with one workgroup instead of two.
//
// A band row that a resident row does not see enters the second product with weight 0.  A tile that
// holds an infinity or a NaN takes a loop over its rows instead, so that what a row does not see
// cannot reach it (0 * inf).
#include "f32_band.hpp"

namespace gformer {
namespace {

template <int D, int QB>
__global__ __launch_bounds__(kF32BandThreads, 2) void windowed_f32_kernel(AttnArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  windowed_f32<D, QB>(a, blockIdx.x, smem_raw);
}
template <int D, int QB>
__global__ __launch_bounds__(kF32BandThreads, 2) void windowed_bwd_q_f32_kernel(BwdArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  windowed_bwd_q_f32<D, QB>(a, blockIdx.x, smem_raw);
}
template <int D, int QB>
__global__ __launch_bounds__(kF32BandThreads, 2) void windowed_bwd_kv_f32_kernel(BwdArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  windowed_bwd_kv_f32<D, QB>(a, blockIdx.x, smem_raw);
}

template <int D, typename Args, typename K4, typename K1>
hipError_t launch_rows(const Args& a, K4 k4, K1 k1, hipStream_t s) {
  const int smem = (int)sizeof(F32WinSmem<D>);
  const int rows = f32_window_rows((int64_t)a.B * a.H0, a.N);
  const dim3 grid((unsigned)((a.N + rows - 1) / rows * a.H0 * a.B)), block(kF32BandThreads);
  hipError_t e;
  if (rows == 64) {
    if ((e = allow_lds(k4, smem)) != hipSuccess) return e;
    k4<<<grid, block, smem, s>>>(a);
  } else {
    if ((e = allow_lds(k1, smem)) != hipSuccess) return e;
    k1<<<grid, block, smem, s>>>(a);
  }
  return hipGetLastError();
}

template <int D> hipError_t launch_bwd(const BwdArgs& a, hipStream_t s) {
  const hipError_t e = launch_rows<D>(a, windowed_bwd_q_f32_kernel<D, 4>, windowed_bwd_q_f32_kernel<D, 1>, s);
  if (e != hipSuccess) return e;
  return launch_rows<D>(a, windowed_bwd_kv_f32_kernel<D, 4>, windowed_bwd_kv_f32_kernel<D, 1>, s);
}

}  // namespace

// 64 rows a workgroup where that gives every compute unit one (12 heads of 2048 rows, 384 workgroups:
// forward 24 against 28 us with 16 rows, dq 48 against 60, dk and dv 37 against 42); below, 16 rows spread
// the call over four times as many.
int f32_window_rows(int64_t heads, int N) {
  return heads * ((N + 63) / 64) >= device_compute_units() ? 64 : 16;
}

hipError_t launch_windowed_f32(const AttnArgs& a, hipStream_t s) {
  if (a.H0 <= 0 || a.N <= 0 || a.B <= 0) return hipSuccess;
  return a.d == 64 ? launch_rows<64>(a, windowed_f32_kernel<64, 4>, windowed_f32_kernel<64, 1>, s)
                   : launch_rows<128>(a, windowed_f32_kernel<128, 4>, windowed_f32_kernel<128, 1>, s);
}

hipError_t launch_windowed_backward_f32(const BwdArgs& a, hipStream_t s) {
  if (a.H0 <= 0 || a.N <= 0 || a.B <= 0) return hipSuccess;
  return a.d == 64 ? launch_bwd<64>(a, s) : launch_bwd<128>(a, s);
}

}  // namespace gformer
