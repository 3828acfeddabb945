// Windowed softmax attention heads on bf16 matrix cores (section III-B, Eq. 1): the causal window
// ending at the token, or (bidirectional variant) the window centred on it.
//
// The query-block kernel: used for windows wider than five key tiles and for small calls (the
// streaming kernel in windowed_stream.hip takes the rest).
//
// One workgroup (4 waves) owns 128 consecutive queries of one (batch, head); each wave owns 32
// of them.  The band of keys those queries can see is walked in tiles of 64 keys; tiles outside
// the band are never touched.  K and V tiles sit in LDS row-major, shared by the 4 waves; K is
// read with 128-bit loads (contraction over the head dimension), V with the LDS transpose
// read (contraction over keys).
//
// Per tile and wave:  S^T = K Q^T  (keys x queries, so one lane owns one query column and the
// running max / sum / rescale are lane-local apart from one exchange between lane l and l^32),
// online softmax in base 2, then O^T += V^T P^T with P^T taken straight from the score
// registers.  Only tiles cut by the diagonal or the window edge are masked.
//
// The K tiles run one step ahead of the V tiles: a step first turns the scores of tile t (made
// at the end of the step before) into weights, which is vector work only, and then issues the
// value products of tile t and the score products of tile t+1 back to back, sixteen and sixteen
// matrix instructions over six independent accumulators with their LDS operands fetched ahead.
// So a wave alternates between a stretch that needs only the vector unit and a stretch that
// needs only the matrix core and LDS, and the two waves a SIMD holds fill each other's gaps.
#include "windowed_block.hpp"

namespace gformer {
namespace {

template <int D, bool NEG>
__global__ __launch_bounds__(kMfmaWindowThreads, 2) void windowed_mfma_kernel(AttnArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  windowed_block<D, NEG>(a, blockIdx.x, smem_raw);
}

}  // namespace

hipError_t launch_windowed_mfma(const AttnArgs& a, hipStream_t s) {
  if (a.H0 <= 0 || a.N <= 0 || a.B <= 0) return hipSuccess;
  dim3 grid(((a.N + BR - 1) / BR) * a.H0 * a.B);
  dim3 block(kMfmaWindowThreads);
  const bool neg = a.scale < 0.f;
  hipError_t e = hipSuccess;
  auto launch = [&](auto kern, int smem) {
    e = allow_lds(kern, smem);
    if (e == hipSuccess) kern<<<grid, block, smem, s>>>(a);
  };
  if (a.d == 64) {
    if (neg) launch(windowed_mfma_kernel<64, true>, (int)sizeof(WinSmem<64>));
    else launch(windowed_mfma_kernel<64, false>, (int)sizeof(WinSmem<64>));
  } else {
    if (neg) launch(windowed_mfma_kernel<128, true>, (int)sizeof(WinSmem<128>));
    else launch(windowed_mfma_kernel<128, false>, (int)sizeof(WinSmem<128>));
  }
  if (e != hipSuccess) return e;
  return hipGetLastError();
}

}  // namespace gformer
