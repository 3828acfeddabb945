// Positive random features as a pre-map of Q or K for the linear heads (section III-A names
// them, Algorithm 1 calls them "random feature maps"; the formula is the construction of the
// work they cite):
//     out[t][i] = exp(w_i . x_t - |x_t|^2 / 2) / sqrt(m),   i = 0..m-1,  m = d here.
// The mapped tensor is then given to the attention call with the identity feature map.
//
// bf16 kernel: one GEMM tile of 32 tokens per wave on the matrix cores, computed transposed,
//     C^T[feature][token] = W X^T,
// so that a lane owns one token: its half of the squared norm comes from the very registers it
// feeds the matrix cores with, and exponent, scaling and rounding are lane-local.  Rows come and go as
// whole rows, 16 bytes a lane, and change to operand layout in the wave's own piece of LDS; the next
// unit's rows are loaded while this one is mapped, and no wave waits for another.  W sits in LDS for the
// lifetime of the workgroup, at d = 64 in registers.
// HBM-bound: 2*d*2 bytes per token-head against 2*d*m FLOP.  Loads in operand layout touch 32 rows an
// instruction, 32 bytes each, and took the memory pipeline with them.  us before, now (same bits):
// 4 x 13 heads x 4096 x 64 14.8, 11.5 (4.75 TB/s); 8 x 10 x 4096 x 64 20.2, 15.8; 2 x 26 x 8192 x 128 49.0, 40.2
// (5.4 TB/s); a call of 1 x 10 x 2048 x 64 is host bound (7.5) as before.
#include "common.hpp"
#include "mfma.hpp"

namespace gformer {
namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kFeatThreads = 256;
constexpr int kFeatWaves = kFeatThreads / 64;
constexpr int kFeatRows = 32;    // tokens of a unit: one wave's tile

template <int D> struct FeatSmem {
  static constexpr int WROW = D + 8;    // row stride = 4 dwords mod 64: conflict-free b128 reads
  static constexpr int OROW = D + 8;
  uint16_t w[D * WROW];                             // W, row-major [feature][input]
  uint16_t ot[kFeatWaves][kFeatRows * OROW];        // a wave's finished rows on their way to memory
};

template <int D>
__global__ __launch_bounds__(kFeatThreads, D == 64 ? 4 : 2) void random_features_mfma_kernel(FeatureArgs a) {
  constexpr int KS = D / 16, NT = D / 32;
  using Smem = FeatSmem<D>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  Smem& sm = *reinterpret_cast<Smem*>(smem_raw);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ln = lane & 31, lh = lane >> 5;
  const int N = a.N, heads = a.head_end - a.head_begin;
  const int per_head = (N + kFeatRows - 1) / kFeatRows, total = a.B * heads * per_head;
  const int step = (int)gridDim.x * kFeatWaves;

  struct Unit {
    int t0;
    const uint16_t* x;
    uint16_t* out;
  };
  auto unit = [&](int u) {
    const int head = u / per_head, b = head / heads, h = a.head_begin + head % heads;
    return Unit{(u - head * per_head) * kFeatRows,
                reinterpret_cast<const uint16_t*>(a.x.base) + b * a.x.sb + h * a.x.sh,
                reinterpret_cast<uint16_t*>(a.out) + b * a.osb + h * a.osh};
  };
  // A unit's rows, 16 bytes a lane and whole rows together; rows past N-1 re-read row N-1 (of the same unit)
  constexpr int C8 = D / 8, PIECES = kFeatRows * C8 / 64;
  const int row = lane / C8, col = 8 * (lane % C8);
  struct Rows { u32x4 x[PIECES]; };
  auto load = [&](Rows& r, const Unit& un) {
#pragma unroll
    for (int i = 0; i < PIECES; ++i)
      r.x[i] = __builtin_nontemporal_load(
          reinterpret_cast<const u32x4*>(un.x + (int64_t)min(un.t0 + row + i * (64 / C8), N - 1) * a.x.sn + col));
  };

  int u = blockIdx.x * kFeatWaves + wave;
  Unit cur = unit(min(u, total - 1));
  Rows rows;
  load(rows, cur);   // on its way while W is staged
  const uint16_t* wp = reinterpret_cast<const uint16_t*>(a.w);
  for (int c = tid; c < D * C8; c += kFeatThreads) {
    const int wrow = c / C8, wcol = 8 * (c % C8);
    *reinterpret_cast<u32x4*>(&sm.w[wrow * Smem::WROW + wcol]) =
        *reinterpret_cast<const u32x4*>(wp + (int64_t)wrow * D + wcol);
  }
  lds_barrier();
  if (u >= total) return;   // uniform over the wave; no barrier follows
  auto w_at = [&](int nt, int ks) { return lds_read16(&sm.w[(32 * nt + ln) * Smem::WROW + 16 * ks + 8 * lh]); };
  constexpr bool HELD = D == 64;   // W in registers: 32 at d = 64, 128 at d = 128
  bf16x8 wr[HELD ? NT * KS : 1];
  if constexpr (HELD) {
#pragma unroll
    for (int x = 0; x < NT * KS; ++x) wr[x] = w_at(x / KS, x % KS);
  }
  // exp(acc - |x|^2/2) / sqrt(m) = 2^((acc - |x|^2/2) * log2(e) - log2(m)/2)
  const float shift = 0.5f * __log2f((float)D);
  uint16_t* const ot = sm.ot[wave];

  auto stage = [&](const Rows& r) {
#pragma unroll
    for (int i = 0; i < PIECES; ++i)
      *reinterpret_cast<u32x4*>(&ot[(row + i * (64 / C8)) * Smem::OROW + col]) = r.x[i];
    wave_sync();   // the rows are this wave's own
  };
  auto map = [&](const Unit& un) {
    bf16x8 xb[KS];   // lane = token
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) xb[ks] = lds_read16(&ot[ln * Smem::OROW + 16 * ks + 8 * lh]);
    // half of |x|^2 from this lane's share of the row, the other half from lane ^ 32
    float sq = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const u32x4 x = as_u32x4(xb[ks]);
#pragma unroll
      for (int i = 0; i < 4; ++i) sq = dot2_bf16(x[i], x[i], sq);
    }
    sq += __shfl_xor(sq, 32, 64);
    const float bias = -(0.5f * sq) * kLog2e - shift;

    f32x16 acc[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[nt][i] = 0.f;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        bf16x8 wa;
        if constexpr (HELD) wa = wr[nt * KS + ks];
        else wa = w_at(nt, ks);
        acc[nt] = mfma32(wa, xb[ks], acc[nt]);
      }
    }
    // register i of tile nt is feature 32*nt + 8*(i/4) + 4*lh + i%4 of this lane's token
    uint16_t* orow = &ot[ln * Smem::OROW + 4 * lh];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float e[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) e[j] = __builtin_amdgcn_exp2f(fmaf(acc[nt][4 * g + j], kLog2e, bias));
        u32x2 pk;
        pk[0] = pack_bf16(e[0], e[1]);
        pk[1] = pack_bf16(e[2], e[3]);
        *reinterpret_cast<u32x2*>(orow + 32 * nt + 8 * g) = pk;
      }
    }
    wave_sync();
#pragma unroll
    for (int i = 0; i < PIECES; ++i) {
      const int at = row + i * (64 / C8);
      if (un.t0 + at < N)
        __builtin_nontemporal_store(*reinterpret_cast<const u32x4*>(&ot[at * Smem::OROW + col]),
                                    reinterpret_cast<u32x4*>(un.out + (int64_t)(un.t0 + at) * a.osn + col));
    }
    wave_sync();   // read before the next unit's rows are staged
  };
  // the next unit's loads are issued without a condition, so that the wait for this unit's leaves them in flight
  for (; u + step < total; u += step) {
    const Unit next = unit(u + step);
    stage(rows);
    load(rows, next);
    map(cur);
    cur = next;
  }
  stage(rows);
  map(cur);
}

// fp32 arithmetic, fp32 or bf16 storage: one workgroup per token, one thread per feature.  The
// row is copied to LDS first, so the map may run in place.
template <typename T>
__global__ __launch_bounds__(128) void random_features_scalar_kernel(FeatureArgs a) {
  __shared__ float xs[128];
  __shared__ float red[128];
  const int d = a.d, N = a.N, heads = a.head_end - a.head_begin;
  const int64_t row = blockIdx.x;                       // over B * heads * N
  const int n = (int)(row % N), hh = (int)((row / N) % heads), b = (int)(row / ((int64_t)N * heads));
  const int h = a.head_begin + hh, i = threadIdx.x;
  const int64_t xo = b * a.x.sb + h * a.x.sh + (int64_t)n * a.x.sn;
  const int64_t oo = b * a.osb + h * a.osh + (int64_t)n * a.osn;
  float v = 0.f;
  if (i < d) v = Storage<T>::load(a.x.base, xo + i);
  xs[i] = v;
  red[i] = v * v;
  __syncthreads();
  for (int s = 64; s > 0; s >>= 1) {
    if (i < s) red[i] += red[i + s];
    __syncthreads();
  }
  if (i >= d) return;
  const float half_sq = 0.5f * red[0];
  float dot = 0.f;
  for (int c = 0; c < d; ++c) dot = fmaf(Storage<T>::load(a.w, (int64_t)i * d + c), xs[c], dot);
  Storage<T>::store(a.out, oo + i, expf(dot - half_sq) * rsqrtf((float)d));
}

template <int D> hipError_t launch_mfma_t(const FeatureArgs& a, hipStream_t s) {
  const int heads = a.head_end - a.head_begin;
  const long units = (long)a.B * heads * ((a.N + kFeatRows - 1) / kFeatRows);
  // Workgroups a compute unit: two, and at d = 64 four (LDS and registers hold them) where a wave then has one or two
  // units and the loads of all waves stand in for the prefetch.  us at two, four: 4 x 13 heads x 4096 12.1, 11.5 (two
  // units a wave); 8 x 10 x 4096 15.8, 16.7 (three); 2 x 26 x 8192 19.8, 21.7 (four).  Three and six: no better anywhere.
  const long cus = device_compute_units();
  const long per_cu = D == 64 && units <= 2 * 4 * kFeatWaves * cus ? 4 : 2;
  // every wave the same number of units, but for the last ones
  const long rounds = (units + per_cu * kFeatWaves * cus - 1) / (per_cu * kFeatWaves * cus);
  const int grid = (int)((units + rounds * kFeatWaves - 1) / (rounds * kFeatWaves));
  const int smem = (int)sizeof(FeatSmem<D>);
  hipError_t e = allow_lds(random_features_mfma_kernel<D>, smem);
  if (e != hipSuccess) return e;
  random_features_mfma_kernel<D><<<dim3(grid), dim3(kFeatThreads), smem, s>>>(a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_random_features(const FeatureArgs& a, bool bf16, bool mfma, hipStream_t s) {
  const int heads = a.head_end - a.head_begin;
  if (a.B <= 0 || heads <= 0 || a.N <= 0) return hipSuccess;
  if (mfma) return a.d == 64 ? launch_mfma_t<64>(a, s) : launch_mfma_t<128>(a, s);
  const int64_t rows = (int64_t)a.B * heads * a.N;
  if (bf16) random_features_scalar_kernel<uint16_t><<<dim3((unsigned)rows), dim3(128), 0, s>>>(a);
  else random_features_scalar_kernel<float><<<dim3((unsigned)rows), dim3(128), 0, s>>>(a);
  return hipGetLastError();
}

}  // namespace gformer
