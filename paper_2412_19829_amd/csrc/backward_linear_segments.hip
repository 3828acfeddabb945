// Backward pass of the linear heads on bf16 matrix cores, heads cut into segments (formulas:
// backward_scalar.hip; the causal layer, and the layer over all keys with CAUSAL = false).
//
// Three walks in chunks of 32 tokens, one workgroup of d/16 waves per segment:
//   sums   A = sum phi(k) v^T, Z = sum phi(k) of every segment
//   dq     from the sums of the segments in front:  r_t = A dO_t,  S_tu = phi(q_t).phi(k_u),
//          T_tu = dO_t.v_u (u <= t inside the chunk),  den_t = sum_u S_tu + phi(q_t).Z + eps,
//          c_t = (phi(q_t).r_t + sum_u S_tu T_tu) / den_t^2,
//          dphi(q_t) = r_t / den_t - c_t Z + sum_u (T_tu / den_t - c_t) phi(k_u);
//          leaves (den, c) of every token and the segment's B = sum phi(q) dO^T / den, Y = sum c phi(q)
//   dk,dv  from the sums of the segments behind:  dphi(k_u) = B v_u - Y + sum_t (T_tu / den_t - c_t) phi(q_t),
//          dv_u = B^T phi(k_u) + sum_t S_tu / den_t dO_t
// c needs no read-out of the forward pass: dO_t.num_t is a product of what dphi(q_t) takes anyway.
//
// Wave w owns columns 16w..16w+15 of the carried sums as 16x16 accumulator tiles whose registers,
// packed to bf16, are the operand of the read-out (v_mfma_f32_16x16x32_bf16, K = 32: tiles 2*kk and
// 2*kk + 1 hold rows 32*kk + 8*g + 0..3 and + 4..7 of lane group g, which is that instruction's order
// of k-slots).  So the sums go through LDS for one product alone, dv's, which wants B by value column (kept in registers in
// both orders, updated twice a chunk: 149 against 147 us for a training step of 52 heads x 4096, and dv 2 to 6 % further from 64
// bits); the tiles of a chunk are nearly all a workgroup needs there, and several workgroups share a compute unit and cover
// each other's barriers.
//
// Head size 64.  Measured (us, the scans of backward_linear_mfma.hip and the sweeps of backward_bidir_mfma.hip
// against these): causal, 52 heads x 4096 tokens, 103 + 99 -> 14 (sums) + 6 (scan) + 45 (dq) + 6 + 40 (dk, dv);
// over all keys, 288 heads x 577, 16 + 43 + 25 -> 12 + 35 + 22.  A scan has one workgroup of four waves on a
// compute unit (85 KB of LDS) and five barriers per 64 tokens, here two to three workgroups interleave.
// Traffic 27 MB a tensor: 136 MB and 164 MB, 3.0 and 4.2 TB/s.  At head size 128 a wave's sums take 64 registers:
// two workgroups on a compute unit leave 128 in all, which spills (830 + 565 us on 104 heads x 8192
// against 477 + 481), one leaves each chunk's chain of barriers exposed (452 + 415, plus 105 for the sums);
// chunks in flight (one to three), waves per column block (one or two) and loads issued late were tried
// on both and none beat the scans, which stay there.
//
// Precision: S, T, den, c, Z, Y and the carried sums are fp32; the weights T/den - c, a difference a
// gradient row sums with signs, enter their products as bf16 pairs (high half + rounded remainder), and so do some
// of the carried sums and of phi(q) / den (which and why: launch_linear_backward_segments).
#include <algorithm>
#include <type_traits>

#include "backward_band.hpp"
#include "common.hpp"
#include "mfma.hpp"

namespace gformer {
namespace {

constexpr int SC = 32;       // tokens per chunk
constexpr int TRW = SC + 4;  // row stride (floats) of the fp32 products
constexpr int WRW = SC + 8;  // row stride (bf16) of the weights
constexpr float kLog2e = 1.4426950408889634f;
constexpr int kSegmentsInPlace = kBidirStateSlots;   // up to this many a walk adds up the sums it needs itself
constexpr u32x4 kZero4 = {0u, 0u, 0u, 0u};

typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr f32x4 kZeroF4 = {0.f, 0.f, 0.f, 0.f};

template <int D> struct SegCfg {
  static_assert(D == 64, "row stride, LDS and registers are laid out for d = 64");
  static constexpr int NW = D / 16, NT = 64 * NW;
  static constexpr int R = D + 8;                      // 36 dwords: row and transpose reads
  static constexpr int KS = D / 32;                    // contraction steps over the head size
  static constexpr int XT = D / 16;                    // tiles of a carried sum per wave
  static constexpr int STATE = D * D + D;
};

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ float sum_over_groups(float x) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ f32x4 lds4f(const float* p) { return *reinterpret_cast<const f32x4*>(p); }

// elu(x) + 1 = max(x + 1, min(exp(x), 1)): the clamp rides on v_exp, and v_maximum3 lets a NaN through, which comes in
// x + 1.  A comparison and a select instead: 328.9 against 325.6 us for the backward pass of 208 heads x 4096.
__device__ __forceinline__ float phi_elu1(float x) {
  const float e = __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(x * kLog2e), 0.f, 1.f);
  return __builtin_elementwise_maximum(x + 1.f, e);
}
template <bool ELU1> __device__ __forceinline__ u32x4 map8(u32x4 v) {
  if (!ELU1) return v;
  u32x4 o;
#pragma unroll
  for (int w = 0; w < 4; ++w) o[w] = pack_bf16(phi_elu1(bf16_lo(v[w])), phi_elu1(bf16_hi(v[w])));
  return o;
}
template <bool ELU1> __device__ __forceinline__ float slope_of(float f) {
  if (!ELU1) return 1.f;
  return f > 1.f ? 1.f : f;
}
__device__ __forceinline__ void get4(const uint16_t* p, float (&f)[4]) {
  const u32x2 pk = *reinterpret_cast<const u32x2*>(p);
  f[0] = bf16_lo(pk[0]); f[1] = bf16_hi(pk[0]); f[2] = bf16_lo(pk[1]); f[3] = bf16_hi(pk[1]);
}
__device__ __forceinline__ void put4(uint16_t* p, float a, float b, float c, float d) {
  u32x2 pk;
  pk[0] = pack_bf16(a, b);
  pk[1] = pack_bf16(c, d);
  *reinterpret_cast<u32x2*>(p) = pk;
}
// x as a pair of bf16x8: high halves and rounded remainders
__device__ __forceinline__ void split8(const float (&x)[8], bf16x8& hi, bf16x8& lo) {
  u32x4 h, l;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    h[w] = pack_bf16(x[2 * w], x[2 * w + 1]);
    l[w] = pack_bf16(x[2 * w] - bf16_lo(h[w]), x[2 * w + 1] - bf16_hi(h[w]));
  }
  hi = as_bf16x8(h);
  lo = as_bf16x8(l);
}
__device__ __forceinline__ void widen8(bf16x8 v, float (&x)[8]) {
  const u32x4 u = as_u32x4(v);
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    x[2 * w] = bf16_lo(u[w]);
    x[2 * w + 1] = bf16_hi(u[w]);
  }
}
__device__ __forceinline__ bf16x8 pack8(const float (&x)[8]) {
  u32x4 u;
#pragma unroll
  for (int w = 0; w < 4; ++w) u[w] = pack_bf16(x[2 * w], x[2 * w + 1]);
  return as_bf16x8(u);
}

// Operand along the rows of a tile: lane (g, i) takes row i, columns 32*kk + 8*g .. +7.
__device__ __forceinline__ bf16x8 row8(const uint16_t* row_lane, int kk) { return lds_read16(row_lane + 32 * kk); }
// Operand down the tokens of a tile: lane (g, i) takes column `col` of the pattern, tokens 8*g .. +7.
// `at` points at this lane's corner: (8*g + i/4) rows down, the pattern's column for i%4.
template <int R> __device__ __forceinline__ bf16x8 col8(const uint16_t* at) {
  const u32x2 a = lds_tr4(at), b = lds_tr4(at + 4 * R);
  return as_bf16x8(u32x4{a[0], a[1], b[0], b[1]});
}

// Carried sum of wave w, element [feature][value] of the fp32 array in memory: tile 2*kk + y,
// register r of lane (g, i) is value 32*kk + 8*g + 4*y + r of feature 16*w + i.
template <int D>
__device__ __forceinline__ void add_sum(f32x4 (&s)[D / 16], const float* src, int wave, int g, int i) {
#pragma unroll
  for (int x = 0; x < D / 16; ++x)
    s[x] += *reinterpret_cast<const f32x4*>(src + (16 * wave + i) * D + 32 * (x / 2) + 8 * g + 4 * (x % 2));
}
template <int D> __device__ __forceinline__ void put_sum(const f32x4 (&s)[D / 16], float* dst, int wave, int g, int i) {
#pragma unroll
  for (int x = 0; x < D / 16; ++x)
    *reinterpret_cast<f32x4*>(dst + (16 * wave + i) * D + 32 * (x / 2) + 8 * g + 4 * (x % 2)) = s[x];
}
template <int D> __device__ __forceinline__ void clear(f32x4 (&s)[D / 16]) {
#pragma unroll
  for (int x = 0; x < D / 16; ++x) s[x] = kZeroF4;
}
// out[tb] += s^T applied to rows 16*tb + i of a tile
template <int D>
__device__ __forceinline__ void read_out(f32x4 (&out)[2], const f32x4 (&s)[D / 16], const uint16_t* rows_lane) {
  constexpr int R = SegCfg<D>::R;
#pragma unroll
  for (int kk = 0; kk < D / 32; ++kk) {
    u32x4 a;
    a[0] = pack_bf16(s[2 * kk][0], s[2 * kk][1]);
    a[1] = pack_bf16(s[2 * kk][2], s[2 * kk][3]);
    a[2] = pack_bf16(s[2 * kk + 1][0], s[2 * kk + 1][1]);
    a[3] = pack_bf16(s[2 * kk + 1][2], s[2 * kk + 1][3]);
    const bf16x8 sa = as_bf16x8(a);
    out[0] = mfma16(sa, row8(rows_lane, kk), out[0]);
    out[1] = mfma16(sa, row8(rows_lane + 16 * R, kk), out[1]);
  }
}
// The same with the sum as a bf16 pair.
template <int D>
__device__ __forceinline__ void read_out_pair(f32x4 (&out)[2], const f32x4 (&s)[D / 16], const uint16_t* rows_lane) {
  constexpr int R = SegCfg<D>::R;
#pragma unroll
  for (int kk = 0; kk < D / 32; ++kk) {
    const float x[8] = {s[2 * kk][0], s[2 * kk][1], s[2 * kk][2], s[2 * kk][3],
                        s[2 * kk + 1][0], s[2 * kk + 1][1], s[2 * kk + 1][2], s[2 * kk + 1][3]};
    bf16x8 hi, lo;
    split8(x, hi, lo);
    const bf16x8 b0 = row8(rows_lane, kk), b1 = row8(rows_lane + 16 * R, kk);
    out[0] = mfma16(hi, b0, out[0]);
    out[1] = mfma16(hi, b1, out[1]);
    out[0] = mfma16(lo, b0, out[0]);
    out[1] = mfma16(lo, b1, out[1]);
  }
}
// s += sum over the chunk's tokens of (row of a tile)^T (x) `col`
template <int D>
__device__ __forceinline__ void add_outer(f32x4 (&s)[D / 16], const uint16_t* wide_lane, bf16x8 col) {
#pragma unroll
  for (int x = 0; x < D / 16; ++x) {
    s[x] = mfma16(col8<SegCfg<D>::R>(wide_lane + 32 * (x / 2) + 4 * (x % 2)), col, s[x]);
    if (x % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // operands of four tiles in flight, not of all: registers
  }
}
// The same with `col` as a bf16 pair.
template <int D>
__device__ __forceinline__ void add_outer_pair(f32x4 (&s)[D / 16], const uint16_t* wide_lane, const float (&col)[8]) {
  bf16x8 hi, lo;
  split8(col, hi, lo);
#pragma unroll
  for (int x0 = 0; x0 < D / 16; x0 += 4) {
    bf16x8 w[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) w[x] = col8<SegCfg<D>::R>(wide_lane + 32 * ((x0 + x) / 2) + 4 * (x % 2));
#pragma unroll
    for (int x = 0; x < 4; ++x) s[x0 + x] = mfma16(w[x], hi, s[x0 + x]);
#pragma unroll
    for (int x = 0; x < 4; ++x) s[x0 + x] = mfma16(w[x], lo, s[x0 + x]);
    __builtin_amdgcn_sched_barrier(0);
  }
}
// 16x16 tile of products of rows
template <int D> __device__ __forceinline__ f32x4 rows_product(const uint16_t* a_lane, const uint16_t* b_lane) {
  f32x4 acc = kZeroF4;
#pragma unroll
  for (int kk = 0; kk < D / 32; ++kk) acc = mfma16(row8(a_lane, kk), row8(b_lane, kk), acc);
  return acc;
}

// Whole chunks run as body(t0, true_type), without a condition in front of their loads and stores: with
// one the compiler waits for everything outstanding, the last stores included, before it stages a
// chunk.  Loads past the end are clamped to the last row.  On the way down a chunk also stores the rows of the one
// before it, so the first one, which has none to store, runs as body(t0, false_type), and so does the
// one that stores a ragged chunk's.
template <typename Body> __device__ __forceinline__ void walk_up(int begin, int end, Body body) {
  int t0 = begin;
  for (; t0 + SC <= end; t0 += SC) body(t0, std::true_type{});
  if (t0 < end) body(t0, std::false_type{});
}
template <typename Body> __device__ __forceinline__ void walk_down(int begin, int end, Body body) {
  int t0 = begin + (end - begin - 1) / SC * SC;
  for (int general = t0 + SC > end ? 2 : 1; general > 0 && t0 >= begin; --general, t0 -= SC) body(t0, std::false_type{});
  for (; t0 >= begin; t0 -= SC) body(t0, std::true_type{});
}

// What every walk knows about its thread.
template <int D> struct Seat {
  int tid, lane, g, i, wave;
  int row, col;                 // the 16-byte piece of a chunk this thread moves
  int seg, head, b, h, begin, end, total;   // tokens [begin, end) in `total` chunks
  int row_at, own_at, wide_at;  // lane corners: rows; own columns down the tokens; all columns down the tokens
  __device__ __forceinline__ Seat(const BwdArgs& a, int block, int segments) {
    constexpr int R = SegCfg<D>::R;
    tid = threadIdx.x;
    lane = tid & 63;
    g = lane >> 4;
    i = lane & 15;
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    row = tid / (D / 8);
    col = 8 * (tid % (D / 8));
    seg = block % segments;
    head = block / segments;
    const int H1 = a.H - a.H0;
    b = head / H1;
    h = a.H0 + head % H1;
    begin = seg * a.lin_segment_len;
    end = min(a.N, begin + a.lin_segment_len);
    total = (end - begin + SC - 1) / SC;
    row_at = i * R + 8 * g;
    own_at = (8 * g + (i >> 2)) * R + 16 * wave + 4 * (i & 3);
    wide_at = (8 * g + (i >> 2)) * R + 8 * (i & 3);
  }
};
// One tensor as a thread moves it: a piece of a chunk is a wave-uniform base and a 32-bit offset that never changes,
// under one clamp (rows past the end re-read the last).  As a 64-bit product per piece, four quarter-rate multiplies, the
// walks took 185.1 in place of 182.2 us (8 x (2 + 10) x 4096, window 256), 116.1 in place of 115.2 (64 heads x 4096).
template <int D> struct Piece {
  uint32_t off, colb;
  int sn;
  __device__ __forceinline__ Piece(const Seat<D>& s, int64_t row_stride)
      : off(2u * (uint32_t)(s.row * (int)row_stride + s.col)), colb(2u * (uint32_t)s.col), sn((int)row_stride) {}
  __device__ __forceinline__ u32x4 load(const uint16_t* head, int t0, int N) const {
    t0 = min(t0, N - 1);
    const uint32_t lim = 2u * (uint32_t)(min(N - 1 - t0, SC - 1) * sn) + colb;
    return *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(head + (int64_t)t0 * sn) + (size_t)min(off, lim));
  }
  __device__ __forceinline__ void store(uint16_t* head, int t0, u32x4 x) const {
    *reinterpret_cast<u32x4*>(reinterpret_cast<char*>(head + (int64_t)t0 * sn) + (size_t)off) = x;
  }
};
template <int D> __device__ __forceinline__ const uint16_t* head_of(const TensorView& t, int b, int h) {
  return reinterpret_cast<const uint16_t*>(t.base) + b * t.sb + h * t.sh;
}

// ---- sums of every segment --------------------------------------------------------------------
template <int D> struct SegSumSmem {
  uint16_t fk[2][SC * SegCfg<D>::R], vv[2][SC * SegCfg<D>::R];
};
template <int D, bool ELU1>
__device__ __forceinline__ void seg_sum(const BwdArgs& a, int block, unsigned char* smem_raw) {
  using C = SegCfg<D>;
  constexpr int R = C::R;
  SegSumSmem<D>& sm = *reinterpret_cast<SegSumSmem<D>*>(smem_raw);
  // segments summed per head: all, or (causal) all but the last
  const Seat<D> s(a, block, a.causal ? a.lin_segments - 1 : a.lin_segments);
  const int N = a.N;
  const uint16_t* kp = head_of<D>(a.k, s.b, s.h);
  const uint16_t* vp = head_of<D>(a.v, s.b, s.h);
  f32x4 acc[C::XT];
  clear<D>(acc);
  float z = 0.f;
  const Piece<D> pk(s, a.k.sn), pv(s, a.v.sn);
  u32x4 kr = pk.load(kp, s.begin, N), vr = pv.load(vp, s.begin, N);
  int it = 0;
  walk_up(s.begin, s.end, [&](int t0, auto) {
    const bool valid = t0 + s.row < N;
    uint16_t *fkt = sm.fk[it & 1], *vvt = sm.vv[it & 1];   // one barrier a chunk: two buffers
    ++it;
    *reinterpret_cast<u32x4*>(fkt + s.row * R + s.col) = valid ? map8<ELU1>(kr) : kZero4;
    *reinterpret_cast<u32x4*>(vvt + s.row * R + s.col) = valid ? vr : kZero4;
    kr = pk.load(kp, t0 + SC, N);
    vr = pv.load(vp, t0 + SC, N);
    lds_barrier();
    const bf16x8 kc = col8<R>(fkt + s.own_at);
    add_outer<D>(acc, vvt + s.wide_at, kc);
    const u32x4 u = as_u32x4(kc);
#pragma unroll
    for (int w = 0; w < 4; ++w) z = dot2_ones_bf16(u[w], z);
  });
  float* dst = a.ws_state + ((int64_t)s.head * a.lin_segments + s.seg) * C::STATE;
  put_sum<D>(acc, dst, s.wave, s.g, s.i);
  z = sum_over_groups(z);
  if (s.g == 0) dst[D * D + 16 * s.wave + s.i] = z;
}

// ---- dq, (den, c), and the segment's B and Y ----------------------------------------------------
// Two barriers a chunk: up to the first, its products; up to the second, what follows from them, the weights of dq (each wave
// makes a quarter for all) and the next chunk's staging into the other buffer; dq itself shares its stretch with
// the next chunk's products.  With one buffer, a barrier more and every wave making all weights for itself the backward
// pass took (us, same bits) 337.2 in place of 328.2 on 208 heads x 4096, 100.8 in place of 99.0 on 52.
template <int D> struct SegQSmem {
  using C = SegCfg<D>;
  struct Tiles {
    uint16_t fq[SC * C::R], fk[SC * C::R], vv[SC * C::R], dd[SC * C::R];
  } buf[2];                      // chunk n in buf[n % 2]
  float t[SC * TRW];             // T, [query][key]
  uint16_t wh[SC * WRW], wl[SC * WRW];   // T / den - c as a pair, [query][key]
  float part[2][3][16];          // row sums of S and of S*T per 16x16 tile
  float red[2][C::NW][SC];       // per-wave parts of phi(q).r and phi(q).Z
  float own[C::NW][2][SC];       // 1/den and c, each wave's own copy
  float z[D];
};
template <int D, bool ELU1, bool CAUSAL, bool PAIR>
__device__ __forceinline__ void seg_q(const BwdArgs& a, int block, unsigned char* smem_raw) {
  using C = SegCfg<D>;
  constexpr int R = C::R, NW = C::NW;
  SegQSmem<D>& sm = *reinterpret_cast<SegQSmem<D>*>(smem_raw);
  const Seat<D> s(a, block, a.lin_segments);
  const int g = s.g, i = s.i, wave = s.wave, N = a.N;
  const uint16_t* qp = head_of<D>(a.q, s.b, s.h);
  const uint16_t* kp = head_of<D>(a.k, s.b, s.h);
  const uint16_t* vp = head_of<D>(a.v, s.b, s.h);
  const uint16_t* dp = head_of<D>(a.dout, s.b, s.h);
  uint16_t* dq = reinterpret_cast<uint16_t*>(a.dq) + s.b * a.q.sb + s.h * a.q.sh;
  float* ws = a.ws + ((int64_t)s.b * a.H + s.h) * N * 2;
  const Piece<D> pq(s, a.q.sn), pk(s, a.k.sn), pv(s, a.v.sn), pd(s, a.dout.sn);
  u32x4 qr, kr = kZero4, vr = kZero4, dr;
  auto load = [&](int t0) {
    qr = pq.load(qp, t0, N);
    dr = pd.load(dp, t0, N);
    if (CAUSAL) {
      kr = pk.load(kp, t0, N);
      vr = pv.load(vp, t0, N);
    }
  };
  load(s.begin);
  f32x4 as[C::XT], bs[C::XT];   // A and this segment's B, columns are features
  clear<D>(as);
  clear<D>(bs);
  float y = 0.f;
  {
    // the sums of the segments in front (all of them over all keys), or their total where a scan ran
    int first = 0, end = CAUSAL ? s.seg : a.lin_segments;
    if (a.lin_segments > kSegmentsInPlace) first = s.seg, end = s.seg + 1;
    float z = 0.f;
    for (int j = first; j < end; ++j) {
      const float* src = a.ws_state + ((int64_t)s.head * a.lin_segments + j) * C::STATE;
      add_sum<D>(as, src, wave, g, i);
      if (s.tid < D) z += src[D * D + s.tid];
    }
    if (s.tid < D) sm.z[s.tid] = z;
  }
  const int piece = s.row * R + s.col;
  auto stage = [&](int n, bool whole) {
    typename SegQSmem<D>::Tiles& b = sm.buf[n & 1];
    const bool valid = whole || s.begin + n * SC + s.row < N;
    *reinterpret_cast<u32x4*>(b.fq + piece) = valid ? map8<ELU1>(qr) : kZero4;
    *reinterpret_cast<u32x4*>(b.dd + piece) = valid ? dr : kZero4;
    if (CAUSAL) {
      *reinterpret_cast<u32x4*>(b.fk + piece) = valid ? map8<ELU1>(kr) : kZero4;
      *reinterpret_cast<u32x4*>(b.vv + piece) = valid ? vr : kZero4;
    }
  };
  auto store_rows = [&](int n, bool all) {   // the chunk's dq rows, left in the phi(q) tile
    const int t0 = s.begin + n * SC;
    if (all || t0 + s.row < N) pq.store(dq, t0, *reinterpret_cast<const u32x4*>(sm.buf[n & 1].fq + piece));
  };
  stage(0, false);
  if (s.total > 1) load(s.begin + SC);
  lds_barrier();
  // Whole chunks between the first and the last but one run as body(n, true_type), without a condition in front of their
  // loads and stores.
  auto body = [&](int n, auto steady) {
    constexpr bool STEADY = decltype(steady)::value;
    const int t0 = s.begin + n * SC;
    typename SegQSmem<D>::Tiles& b = sm.buf[n & 1];
    if (CAUSAL && wave < 3) {
      // S and T of 16 queries and 16 keys: lane = query, registers = keys 4*g + r
      const int tb = wave > 0, ub = wave > 1;
      const f32x4 sv = rows_product<D>(b.fk + 16 * ub * R + s.row_at, b.fq + 16 * tb * R + s.row_at);
      const f32x4 tv = rows_product<D>(b.vv + 16 * ub * R + s.row_at, b.dd + 16 * tb * R + s.row_at);
      *reinterpret_cast<f32x4*>(sm.t + (16 * tb + i) * TRW + 16 * ub + 4 * g) = tv;
      float ss = 0.f, st = 0.f;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        // T is masked as well: a later token's product may be infinite
        const bool seen = tb != ub || 4 * g + r <= i;
        const float x = seen ? sv[r] : 0.f;
        ss += x;
        st = fmaf(x, seen ? tv[r] : 0.f, st);
      }
      ss = sum_over_groups(ss);
      st = sum_over_groups(st);
      if (g == 0) {
        sm.part[0][wave][i] = ss;
        sm.part[1][wave][i] = st;
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    f32x4 rv[2] = {kZeroF4, kZeroF4};
    if constexpr (PAIR) read_out_pair<D>(rv, as, b.dd + s.row_at);
    else read_out<D>(rv, as, b.dd + s.row_at);
    uint16_t* const corner = b.fq + i * R + 16 * wave + 4 * g;   // this wave's columns of token i (and 16 + i)
    const f32x4 zc = lds4f(sm.z + 16 * wave + 4 * g);   // the sum in front of this chunk
    {
#pragma unroll
      for (int tb = 0; tb < 2; ++tb) {
        float qc[4], qr_ = 0.f, qz = 0.f;
        get4(corner + 16 * tb * R, qc);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          qr_ = fmaf(qc[r], rv[tb][r], qr_);
          qz = fmaf(qc[r], zc[r], qz);
        }
        qr_ = sum_over_groups(qr_);
        qz = sum_over_groups(qz);
        if (g == 0) {
          sm.red[0][wave][16 * tb + i] = qr_;
          sm.red[1][wave][16 * tb + i] = qz;
        }
      }
    }
    lds_barrier();   // T and the parts are visible; the chunk before has its dq rows
    float inv[2], cv[2];
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) {
      const int n = t0 + 16 * tb + i;
      float qr_ = 0.f, qz = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        qr_ += sm.red[0][w][16 * tb + i];
        qz += sm.red[1][w][16 * tb + i];
      }
      if (CAUSAL) {
        qz += tb == 0 ? sm.part[0][0][i] : sm.part[0][1][i] + sm.part[0][2][i];
        qr_ += tb == 0 ? sm.part[1][0][i] : sm.part[1][1][i] + sm.part[1][2][i];
      }
      const float den = STEADY || n < N ? qz + a.eps : 1.f;   // rows past the end: dO is zero
      inv[tb] = 1.f / den;
      cv[tb] = qr_ * inv[tb] * inv[tb];
      if (wave == 0 && (STEADY || n < N))   // every wave has the token's values
        *reinterpret_cast<float2*>(ws + 2 * (int64_t)n) = make_float2(den, cv[tb]);
      if (g == 0) {
        sm.own[wave][0][16 * tb + i] = inv[tb];
        sm.own[wave][1][16 * tb + i] = cv[tb];
      }
    }
    if (CAUSAL) {
      // weights of eight queries, four keys a lane
      const int at = 8 * wave + (s.lane >> 3), k0 = 4 * (s.lane & 7);
      const float iv = sm.own[wave][0][at], cq = sm.own[wave][1][at];
      const f32x4 tv = lds4f(sm.t + at * TRW + k0);
      u32x2 h, l;
      float w[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = k0 + e <= at ? fmaf(tv[e], iv, -cq) : 0.f;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        h[e] = pack_bf16(w[2 * e], w[2 * e + 1]);
        l[e] = pack_bf16(w[2 * e] - bf16_lo(h[e]), w[2 * e + 1] - bf16_hi(h[e]));
      }
      *reinterpret_cast<u32x2*>(sm.wh + at * WRW + k0) = h;
      *reinterpret_cast<u32x2*>(sm.wl + at * WRW + k0) = l;
    }
    if (STEADY || n > 0) store_rows(n - 1, true);
    if (STEADY || n + 1 < s.total) stage(n + 1, STEADY);
    if (STEADY || n + 2 < s.total) load(t0 + 2 * SC);
    __builtin_amdgcn_sched_barrier(0);
    {
      // B += phi(q)^T dO / den, Y += c phi(q): 1/den and c of tokens 8*g .. +7
      float qx[8];
      widen8(col8<R>(b.fq + s.own_at), qx);
      const float* ip = sm.own[wave][0] + 8 * g;
      const float* cp = sm.own[wave][1] + 8 * g;
      const f32x4 i0 = lds4f(ip), i1 = lds4f(ip + 4), c0 = lds4f(cp), c1 = lds4f(cp + 4);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        y = fmaf(j < 4 ? c0[j % 4] : c1[j % 4], qx[j], y);
        qx[j] *= j < 4 ? i0[j % 4] : i1[j % 4];
      }
      if constexpr (CAUSAL) {
        add_outer<D>(bs, b.dd + s.wide_at, pack8(qx));
      } else {
        // over all keys dphi(k) = B v - Y cancels on heads of a few tokens: phi(q) / den as a pair
        add_outer_pair<D>(bs, b.dd + s.wide_at, qx);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 kc;
    if (CAUSAL) {
      kc = col8<R>(b.fk + s.own_at);
      add_outer<D>(as, b.vv + s.wide_at, kc);
      const u32x4 u = as_u32x4(kc);
      float dz = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) dz = dot2_ones_bf16(u[w], dz);
      dz = sum_over_groups(dz);
      if (g == 0) sm.z[16 * wave + i] += dz;   // read by this wave alone
    }
    lds_barrier();   // the weights are visible, the next chunk is staged
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) {
      f32x4 acc;
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[r] = rv[tb][r] * inv[tb] - cv[tb] * zc[r];
      if (CAUSAL) {
        const int off = (16 * tb + i) * WRW + 8 * g;
        acc = mfma16(kc, lds_read16(sm.wh + off), acc);
        acc = mfma16(kc, lds_read16(sm.wl + off), acc);
      }
      float qc[4];
      get4(corner + 16 * tb * R, qc);
      put4(corner + 16 * tb * R, acc[0] * slope_of<ELU1>(qc[0]), acc[1] * slope_of<ELU1>(qc[1]),
           acc[2] * slope_of<ELU1>(qc[2]), acc[3] * slope_of<ELU1>(qc[3]));
    }
  };
  int n = 0;
  body(n++, std::false_type{});
  for (; n + 2 < s.total; ++n) body(n, std::true_type{});
  for (; n < s.total; ++n) body(n, std::false_type{});
  lds_barrier();
  store_rows(s.total - 1, false);
  if (CAUSAL && s.seg == 0) return;   // nothing lies in front of a head's first segment
  float* dst = a.ws_state + ((int64_t)a.B * (a.H - a.H0) * a.lin_segments + (int64_t)s.head * a.lin_segments + s.seg) * C::STATE;
  put_sum<D>(bs, dst, wave, g, i);
  y = sum_over_groups(y);
  if (g == 0) dst[D * D + 16 * wave + i] = y;
}

// ---- dk and dv -----------------------------------------------------------------------------------
template <int D> struct SegKvSmem {
  using C = SegCfg<D>;
  uint16_t fq[SC * C::R], fk[SC * C::R], vv[SC * C::R], dd[SC * C::R];
  uint16_t sw[SC * WRW], wh[SC * WRW], wl[SC * WRW];   // S / den and the pair of T / den - c, [key][query]
  uint16_t bt[D * C::R];                               // bf16 copy of B, [feature][value]
  float inv[SC], cc[SC];
  float y[D];
};
template <int D, bool ELU1, bool CAUSAL, bool PAIR>
__device__ __forceinline__ void seg_kv(const BwdArgs& a, int block, unsigned char* smem_raw) {
  using C = SegCfg<D>;
  constexpr int R = C::R, NW = C::NW;
  SegKvSmem<D>& sm = *reinterpret_cast<SegKvSmem<D>*>(smem_raw);
  const Seat<D> s(a, block, a.lin_segments);
  const int g = s.g, i = s.i, wave = s.wave, N = a.N;
  const uint16_t* qp = head_of<D>(a.q, s.b, s.h);
  const uint16_t* kp = head_of<D>(a.k, s.b, s.h);
  const uint16_t* vp = head_of<D>(a.v, s.b, s.h);
  const uint16_t* dp = head_of<D>(a.dout, s.b, s.h);
  uint16_t* dk = reinterpret_cast<uint16_t*>(a.dk) + s.b * a.k.sb + s.h * a.k.sh;
  uint16_t* dv = reinterpret_cast<uint16_t*>(a.dv) + s.b * a.v.sb + s.h * a.v.sh;
  const float* ws = a.ws + ((int64_t)s.b * a.H + s.h) * N * 2;
  const Piece<D> pq(s, a.q.sn), pk(s, a.k.sn), pv(s, a.v.sn), pd(s, a.dout.sn);
  u32x4 qr = kZero4, kr, vr, dr = kZero4;
  float2 stat = {1.f, 0.f};
  auto load = [&](int t0) {   // walking down: chunks in front of the segment are not read
    t0 = max(t0, s.begin);
    kr = pk.load(kp, t0, N);
    vr = pv.load(vp, t0, N);
    if (CAUSAL) {
      qr = pq.load(qp, t0, N);
      dr = pd.load(dp, t0, N);
      stat = *reinterpret_cast<const float2*>(ws + 2 * (int64_t)min(t0 + (s.tid & (SC - 1)), N - 1));
    }
  };
  const int last = s.begin + (s.total - 1) * SC;
  load(last);
  f32x4 b1[C::XT];   // B, columns are features: dk's operand; dv takes it by value column, from a copy in LDS
  clear<D>(b1);
  {
    int first = CAUSAL ? s.seg + 1 : 0, end = a.lin_segments;   // the segments behind, or their total
    if (a.lin_segments > kSegmentsInPlace) first = s.seg, end = s.seg + 1;
    float yz = 0.f;
    for (int j = first; j < end; ++j) {
      const float* src = a.ws_state + ((int64_t)(a.B * (a.H - a.H0) + s.head) * a.lin_segments + j) * C::STATE;
      add_sum<D>(b1, src, wave, g, i);
      if (s.tid < D) yz += src[D * D + s.tid];
    }
    if (s.tid < D) sm.y[s.tid] = yz;
  }
  auto copy_b = [&]() {
#pragma unroll
    for (int x = 0; x < C::XT; ++x)
      put4(sm.bt + (16 * wave + i) * R + 32 * (x / 2) + 8 * g + 4 * (x % 2), b1[x][0], b1[x][1], b1[x][2], b1[x][3]);
  };
  copy_b();
  uint16_t* const piece_k = sm.fk + s.row * R + s.col;
  uint16_t* const piece_v = sm.vv + s.row * R + s.col;
  auto store_rows = [&](int t0, bool all) {
    if (all || t0 + s.row < N) {
      pk.store(dk, t0, *reinterpret_cast<const u32x4*>(piece_k));
      pv.store(dv, t0, *reinterpret_cast<const u32x4*>(piece_v));
    }
  };
  walk_down(s.begin, s.end, [&](int t0, auto steady) {
    constexpr bool STEADY = decltype(steady)::value;
    lds_barrier();   // the chunk before is consumed, its dk and dv rows are complete
    if (STEADY || t0 < last) store_rows(t0 + SC, STEADY || t0 + 2 * SC <= N);
    const bool valid = STEADY || t0 + s.row < N;
    *reinterpret_cast<u32x4*>(piece_k) = valid ? map8<ELU1>(kr) : kZero4;
    *reinterpret_cast<u32x4*>(piece_v) = valid ? vr : kZero4;
    if (CAUSAL) {
      *reinterpret_cast<u32x4*>(sm.fq + s.row * R + s.col) = valid ? map8<ELU1>(qr) : kZero4;
      *reinterpret_cast<u32x4*>(sm.dd + s.row * R + s.col) = valid ? dr : kZero4;
      if (s.tid < SC) {
        const bool there = STEADY || t0 + s.tid < N;
        sm.inv[s.tid] = there ? 1.f / stat.x : 1.f;
        sm.cc[s.tid] = there ? stat.y : 0.f;
      }
    }
    load(t0 - SC);
    lds_barrier();
    if (CAUSAL) {
      // S / den and T / den - c of 16 keys and 16 queries: lane = key, registers = queries 4*g + r
      for (int x = wave; x < 6; x += NW) {
        const int t = x % 3, ub = t > 1, tb = t > 0;
        const f32x4 inv = lds4f(sm.inv + 16 * tb + 4 * g);
        const int at = (16 * ub + i) * WRW + 16 * tb + 4 * g;
        float w[4];
        if (x < 3) {
          const f32x4 p = rows_product<D>(sm.fq + 16 * tb * R + s.row_at, sm.fk + 16 * ub * R + s.row_at);
#pragma unroll
          for (int r = 0; r < 4; ++r) w[r] = (tb != ub || 4 * g + r >= i) ? p[r] * inv[r] : 0.f;
          put4(sm.sw + at, w[0], w[1], w[2], w[3]);
        } else {
          const f32x4 p = rows_product<D>(sm.dd + 16 * tb * R + s.row_at, sm.vv + 16 * ub * R + s.row_at);
          const f32x4 c = lds4f(sm.cc + 16 * tb + 4 * g);
          u32x2 h, l;
#pragma unroll
          for (int r = 0; r < 4; ++r) w[r] = (tb != ub || 4 * g + r >= i) ? fmaf(p[r], inv[r], -c[r]) : 0.f;
          h[0] = pack_bf16(w[0], w[1]);
          h[1] = pack_bf16(w[2], w[3]);
          l[0] = pack_bf16(w[0] - bf16_lo(h[0]), w[1] - bf16_hi(h[0]));
          l[1] = pack_bf16(w[2] - bf16_lo(h[1]), w[3] - bf16_hi(h[1]));
          *reinterpret_cast<u32x2*>(sm.wh + at) = h;
          *reinterpret_cast<u32x2*>(sm.wl + at) = l;
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    const f32x4 yc = lds4f(sm.y + 16 * wave + 4 * g);
    f32x4 dka[2] = {-yc, -yc}, dva[2] = {kZeroF4, kZeroF4};
    read_out_pair<D>(dka, b1, sm.vv + s.row_at);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < C::KS; ++kk) {
      const bf16x8 bv = col8<R>(sm.bt + 32 * kk * R + s.own_at);
      dva[0] = mfma16(bv, row8(sm.fk + s.row_at, kk), dva[0]);
      dva[1] = mfma16(bv, row8(sm.fk + s.row_at + 16 * R, kk), dva[1]);
    }
    bf16x8 qcol, dcol;
    lds_barrier();   // weights visible; every row read of the phi(k) and v tiles is done
    if (CAUSAL) {
      qcol = col8<R>(sm.fq + s.own_at);
      dcol = col8<R>(sm.dd + s.own_at);
#pragma unroll
      for (int ub = 0; ub < 2; ++ub) {
        const int off = (16 * ub + i) * WRW + 8 * g;
        // the tile of queries 0..15 and keys 16..31 is never written: its weights are zero
        const bool none = ub == 1 && g < 2;
        const bf16x8 h = as_bf16x8(none ? kZero4 : as_u32x4(lds_read16(sm.wh + off)));
        const bf16x8 l = as_bf16x8(none ? kZero4 : as_u32x4(lds_read16(sm.wl + off)));
        const bf16x8 p = as_bf16x8(none ? kZero4 : as_u32x4(lds_read16(sm.sw + off)));
        dka[ub] = mfma16(qcol, h, dka[ub]);
        dva[ub] = mfma16(dcol, p, dva[ub]);
        dka[ub] = mfma16(qcol, l, dka[ub]);
      }
    }
#pragma unroll
    for (int ub = 0; ub < 2; ++ub) {
      uint16_t* kat = sm.fk + (16 * ub + i) * R + 16 * wave + 4 * g;   // this wave's own corner
      float f[4];
      get4(kat, f);
      put4(kat, dka[ub][0] * slope_of<ELU1>(f[0]), dka[ub][1] * slope_of<ELU1>(f[1]),
           dka[ub][2] * slope_of<ELU1>(f[2]), dka[ub][3] * slope_of<ELU1>(f[3]));
      put4(sm.vv + (16 * ub + i) * R + 16 * wave + 4 * g, dva[ub][0], dva[ub][1], dva[ub][2], dva[ub][3]);
    }
    if (CAUSAL) {
      const f32x4 i0 = lds4f(sm.inv + 8 * g), i1 = lds4f(sm.inv + 8 * g + 4);
      const f32x4 c0 = lds4f(sm.cc + 8 * g), c1 = lds4f(sm.cc + 8 * g + 4);
      float qx[8], dy = 0.f;
      widen8(qcol, qx);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        dy = fmaf(j < 4 ? c0[j % 4] : c1[j % 4], qx[j], dy);
        qx[j] *= j < 4 ? i0[j % 4] : i1[j % 4];
      }
      if constexpr (PAIR) add_outer_pair<D>(b1, sm.dd + s.wide_at, qx);
      else add_outer<D>(b1, sm.dd + s.wide_at, pack8(qx));
      copy_b();   // last read in front of the barrier above
      dy = sum_over_groups(dy);
      if (g == 0) sm.y[16 * wave + i] += dy;   // read by this wave alone
    }
  });
  lds_barrier();
  store_rows(s.begin, s.begin + SC <= N);
}

// ---- launches --------------------------------------------------------------------------------------
// One walk, and in the same launch the pass over the windowed heads' band that goes with it: blocks
// [0, linear) are the walk's, those from the next multiple of 8 on (the XCDs keep their runs) the band's.
// A walk's few long workgroups leave the chip half empty at their end, a band pass hardly starts before it
// ends; together one fills what the other leaves.  Same bits.  Measured (us a call, forward and backward
// with recording): 16 x (4 + 2 heads) x 1024 tokens x 64, window 128, causal: 219 apart, 182 together;
// 64 x (3 + 3) x 256 bidirectional, window 14: 161 and 139.  One pass for dk and dv (four products a tile in
// place of five, 190 registers, so two workgroups per compute unit): 189 and 145; at three it spills.
enum Walk { kSumWalk, kQWalk, kKvWalk };
template <int D, bool ELU1, bool CAUSAL, bool PAIR, int WALK>
__global__ __launch_bounds__(SegCfg<D>::NT, 3) void linear_seg_kernel(BwdArgs a, int linear, int rows) {
  static_assert(SegCfg<D>::NT == kBandThreads, "one block size for both kinds of workgroup");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  const int block = blockIdx.x, first = (linear + 7) & ~7;
  if (block < linear) {
    if constexpr (WALK == kSumWalk) seg_sum<D, ELU1>(a, block, smem_raw);
    else if constexpr (WALK == kQWalk) seg_q<D, ELU1, CAUSAL, PAIR>(a, block, smem_raw);
    else seg_kv<D, ELU1, CAUSAL, PAIR>(a, block, smem_raw);
  } else if (block >= first) {
    if constexpr (WALK == kSumWalk) windowed_band<D, kStats>(a, block - first, smem_raw);
    else if constexpr (WALK == kQWalk) windowed_band<D, kDq>(a, block - first, smem_raw);
    else if (block < first + rows) windowed_band<D, kDk>(a, block - first, smem_raw);   // the longer pass first
    else if (block >= first + ((rows + 7) & ~7)) windowed_band<D, kDv>(a, block - first - ((rows + 7) & ~7), smem_raw);
  }
}

template <int D, bool ELU1, bool CAUSAL, bool PAIR> hipError_t launch_t(const BwdArgs& a, bool band, hipStream_t s) {
  using C = SegCfg<D>;
  const int heads = a.B * (a.H - a.H0), nseg = a.lin_segments, per_head = CAUSAL ? nseg - 1 : nseg;
  const int rows = band ? (a.N + band_rows(C::NT) - 1) / band_rows(C::NT) * a.H0 * a.B : 0;   // the band's blocks
  float* bsums = a.ws_state + (int64_t)heads * nseg * C::STATE;
  hipError_t e = hipSuccess;
  auto launch = [&](auto kern, size_t smem, int linear, int band_blocks) {
    if (e != hipSuccess || linear + rows == 0) return;
    if (rows > 0 && smem < sizeof(BandSmem<D>)) smem = sizeof(BandSmem<D>);
    e = allow_lds(kern, smem);
    if (e != hipSuccess) return;
    kern<<<dim3(rows > 0 ? ((linear + 7) & ~7) + band_blocks : linear), dim3(C::NT), smem, s>>>(a, linear, rows);
    e = hipGetLastError();
  };
  launch(linear_seg_kernel<D, ELU1, CAUSAL, !CAUSAL, kSumWalk>, sizeof(SegSumSmem<D>), heads * per_head, rows);
  if (e == hipSuccess && nseg > kSegmentsInPlace) e = launch_segment_scan(a.ws_state, heads, nseg, C::STATE, 0, s);
  launch(linear_seg_kernel<D, ELU1, CAUSAL, PAIR, kQWalk>, sizeof(SegQSmem<D>), heads * nseg, rows);
  if (e == hipSuccess && nseg > kSegmentsInPlace) e = launch_segment_scan(bsums, heads, nseg, C::STATE, 1, s);
  launch(linear_seg_kernel<D, ELU1, CAUSAL, PAIR, kKvWalk>, sizeof(SegKvSmem<D>), heads * nseg, ((rows + 7) & ~7) + rows);
  return e;
}

}  // namespace

int64_t backward_band_tiles(int64_t windowed_heads, int N, int wleft, int wright) {
  const int rows = band_rows(kBandThreads);
  const int64_t tiles = std::min(((int64_t)wleft + wright + rows - 1 + BC - 1) / BC + 1, ((int64_t)N + BC - 1) / BC);
  return windowed_heads * ((N + rows - 1) / rows) * tiles;
}

// Three workgroups per compute unit and no segment under 128 tokens: 52 heads of 4096 tokens take 50 + 44 us
// (dq, dk/dv walk) with two, 46 + 40 with three, 51 + 38 with four.  Over all keys a walk reads every sum of
// its head: four segments at most, as many as the workspace of that form has always held.
// A causal call whose band passes weigh half of its walks or more (a tile about one and a half chunks) may get two walks a
// unit: with three there is no room beside them, and the band runs behind them on a chip that empties.  All passes, us,
// three and two a unit, by band's share: 6 x (1 + 7) x 8192, window 128 (0.3) 167.0 and 166.1; 8 x (2 + 10) x 4096, 128
// (0.4) 161.9 and 165.4; 4 x (3 + 13) x 4096, 128 (0.45) 117.2 and 123.0; 8 x (2 + 10) x 4096, 256 (0.55) 180.1 and
// 174.3; 1 x (2 + 10) x 8192, 256 (0.55) 81.5 and 74.9; 16 x (2 + 6) x 1500, 128 (0.65) 101.9 and 96.5; 4 x (5 + 27) x
// 2048, 512 (0.8) 149.0 and 135.4; 8 x (4 + 8) x 2048, 256 (1.3) 122.1 and 115.6; 4 x (8 + 8) x 4096, 256 (2.6) 159.2
// and 156.1.  Up to a share of 4/3 that holds only where the cut into fewer segments is no worse for the fullest unit,
// whose chunks may be an eighth more: with a few heads more than a unit count divides they are a third more, and 12 x
// (8 + 24) x 1024, 128 (0.6) takes 154.1 and 196.9, 22 x (4 + 12) x 2000, 256 (0.9) 304.0 and 374.3, 21 x (3 + 9) x 3297,
// 32 (0.5) 316.0 and 353.3, 15 x (14 + 18) x 2880, 22 (1.2) 530.4 and 597.3; above, 24 x (8 + 8) x 2500, 128 (1.9) 435.4 and
// 416.5.  Nor where a walk is longer than 48 chunks, as the band is gone long before it ends: 8 x (6 + 26) x 4096, 256
// (0.6, 64 chunks) 440.0 and 450.0, x 3000 (47 chunks) 324.1 and 327.9, 16 x (3 + 13) x 2048 (32) 224.6 and 216.7.
Segments backward_segments(int64_t heads, int N, int d, bool causal, int64_t band_tiles) {
  if (heads <= 0 || N <= 0 || d != 64) return Segments{N, 1};
  const int64_t chunks = (N + SC - 1) / SC, most = causal ? kMaxSegments : kBidirStateSlots, cus = device_compute_units();
  auto cut = [&](int walks) {
    const int64_t n = std::min(std::min(walks * cus / heads, most), chunks / 4);
    if (n <= 1) return Segments{N, 1};
    const int len = (int)((chunks + n - 1) / n) * SC;
    return Segments{len, (N + len - 1) / len};
  };
  const Segments three = cut(3);
  if (!causal || 3 * band_tiles < heads * chunks) return three;
  const Segments two = cut(2);
  if (9 * band_tiles >= 8 * heads * chunks) return two;
  auto fullest = [&](const Segments& f) { return (heads * f.count + cus - 1) / cus * ((f.len + SC - 1) / SC); };
  return 8 * fullest(two) <= 9 * fullest(three) && two.len <= 48 * SC ? two : three;
}

// Roundings.  Over all keys, and for causal calls of less than 256 tokens, the sums in the read-outs and phi(q) / den
// in the dk walk are bf16 pairs; longer causal calls have a pair in dk's read-out alone.  A chunk of 32 tokens
// leaves more of a row to the carried sums than the scans' 64 do, whose in-chunk weights are pairs: with one bf16 in
// dk's read-out dk was 3-5 % further from 64 bits than the scans' over all lengths (4096 tokens: 3.15e-3 of its norm
// against 3.06e-3; a pair: 2.86e-3), and short heads need the others as well (100 tokens, dq and dk: scans 4.04e-3 and
// 2.66e-3, one pair 4.08e-3 and 2.68e-3, all 3.82e-3 and 2.55e-3; from 150 on the one is enough).  The pair in the
// read-out costs 1 us of 114 (64 heads x 4096), all of them 6.
hipError_t launch_linear_backward_segments(const BwdArgs& a, bool with_windowed, hipStream_t s) {
  if (a.H - a.H0 <= 0 || a.N <= 0 || a.B <= 0) return hipSuccess;
  const bool elu1 = a.phi == 0;
  if (!a.causal) return elu1 ? launch_t<64, true, false, true>(a, with_windowed, s) : launch_t<64, false, false, true>(a, with_windowed, s);
  if (a.N < 256) return elu1 ? launch_t<64, true, true, true>(a, with_windowed, s) : launch_t<64, false, true, true>(a, with_windowed, s);
  return elu1 ? launch_t<64, true, true, false>(a, with_windowed, s) : launch_t<64, false, true, false>(a, with_windowed, s);
}

}  // namespace gformer
