// Linear heads in single precision on the matrix cores: the causal form (section III-C, Algorithm 1)
// and the form over all keys (section II-B), forward and backward (formulas: backward_scalar.hip).
//
// Chunks of 32 tokens: inside a chunk the masked products, across chunks the carried d x d sum.  A
// workgroup has d/16 waves; wave w owns columns 16w..16w+15 of the carried sum, whose accumulator
// registers are an operand of the read-out as they stand (f32_mfma.hpp), so the sum stays in
// registers for the whole walk.  A head is cut into segments, one workgroup each: a first kernel sums
// every segment by itself, and a walk starts from the sums of the segments before it (backward: of
// the segments behind it too; the dq walk leaves those sums, so Q and dO are not read again for
// them).  One workgroup per head, as the plain-FMA kernels have it, leaves a serial chain of the
// whole sequence on a part of the chip.
//
// Measured, B=4, 52 linear heads, N=2048, d=64, eight segments a head and no scan of their sums (plain-FMA kernels ->
// these, us): forward 1017 -> 17 (sums) + 46, backward 859 + 1558 -> 17 + 68 + 65.  The bound is the SIMDs' issue: the
// matrix core is busy 33 % of the forward walk's time (34 and 39 % of the others'), the vector unit 22 % (24 and 20 %)
// at four cycles an instruction, hardly ever both; with two workgroups a unit the barriers between a chunk's steps
// leave the rest.
//
// Every sum lies in the workspace as A row-major [feature][value], then its vector.
#include <algorithm>
#include <type_traits>

#include "f32_band.hpp"
#include "f32_mfma.hpp"
#include "scalar_util.hpp"
#include "mfma.hpp"

namespace gformer {
namespace {

constexpr int CH = 32;             // tokens per chunk
constexpr int PR = CH + 4;         // row stride of the chunk's masked products
// Up to this many segments a walk adds up the sums it needs itself; beyond, a scan kernel runs first
// (12 segments: 51, 68 and 79 us for the three walks in place, 43 + 7, 61 + 7 and 68 + 7 with the scan).
constexpr int kSumInPlace = 8;

// phi(x) = elu(x) + 1 without a branch (52 against 55 us for the forward walk; written as `x > 0 ? x + 1 : expf(x)` every element gets its own
// jump around the exponential, and the library's expf spends a third of its instructions on ranges
// that do not occur here).  exp(x) = 2^n 2^f with n = round(x log2 e), f = x log2 e - n (Cody and Waite's reduction: log2 e as a
// float and the rest, in fused multiply-adds); v_exp_f32 is good to 1 ulp there and ldexp rounds small
// results once.  A NaN compares false and comes back through x + 1.
__device__ __forceinline__ float elu1_f32(float x) {
  constexpr float kLog2eHi = 1.44269502162933349609375f, kLog2eLo = 1.92596299112661746887e-8f;
  const float c = fmaxf(x, -104.f);   // exp(-104) rounds to 0
  const float n = __builtin_rintf(c * kLog2eHi);
  const float f = fmaf(c, kLog2eLo, fmaf(c, kLog2eHi, -n));
  const float e = __builtin_amdgcn_ldexpf(__builtin_amdgcn_exp2f(f), (int)n);
  return x <= 0.f ? e : x + 1.f;
}

template <int D> constexpr int kLinThreads = 4 * D;   // d/16 waves
template <int D> constexpr int kLinState = D * D + D;

// Maximum over the D/4 consecutive lanes that hold a row: rotations inside 16 lanes, and their neighbours at d = 128.
template <int CTRL> __device__ __forceinline__ float rotated(float x) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), CTRL, 0xf, 0xf, false));
}
template <int D> __device__ __forceinline__ float row_max(float x) {
  x = fmaxf(x, rotated<0x121>(x));
  x = fmaxf(x, rotated<0x122>(x));
  x = fmaxf(x, rotated<0x124>(x));
  x = fmaxf(x, rotated<0x128>(x));
  if (D == 128) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
  return x;
}

// Thread t moves 16-byte pieces (rows t / (D/4) and 16 further on) of a chunk.
template <int D> struct Rows {
  static constexpr int TR = kF32Row<D>;
  int row, col;
  __device__ __forceinline__ explicit Rows(int tid) : row(tid / (D / 4)), col(4 * (tid % (D / 4))) {}
  // rows past the end are stored as zeros: they contribute nothing
  __device__ __forceinline__ void store(float* tile, const f32x4 (&x)[2], int t0, int N) const {
#pragma unroll
    for (int p = 0; p < 2; ++p)
      *reinterpret_cast<f32x4*>(tile + (row + 16 * p) * TR + col) = t0 + row + 16 * p < N ? x[p] : kZeroF4;
  }
  // ... each row divided by the power of two its largest magnitude lies in [1, 2) of; exps[row] receives the
  // exponent.  A row of zeros (or with an infinity) stays as it is, with some exponent that does no harm.
  __device__ __forceinline__ void store_normalised(float* tile, const f32x4 (&x)[2], int* exps, int t0, int N) const {
    f32x4 y[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const float m = row_max<D>(fmaxf(fmaxf(fabsf(x[p][0]), fabsf(x[p][1])), fmaxf(fabsf(x[p][2]), fabsf(x[p][3]))));
      const int e = __builtin_amdgcn_frexp_expf(m) - 1;
#pragma unroll
      for (int j = 0; j < 4; ++j) y[p][j] = __builtin_amdgcn_ldexpf(x[p][j], -e);
      if (col == 0) exps[row + 16 * p] = e;
    }
    store(tile, y, t0, N);
  }
  __device__ __forceinline__ void store_mapped(float* tile, const f32x4 (&x)[2], int t0, int N, int phi) const {
    f32x4 f[2] = {x[0], x[1]};
    if (phi == 0) {   // uniform
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int j = 0; j < 4; ++j) f[p][j] = elu1_f32(x[p][j]);
    }
    store(tile, f, t0, N);
  }
};

// One tensor as a thread reads it: a wave-uniform base and a 32-bit offset that never changes, under one clamp (rows
// past the end re-read the last, in bounds).  As a 64-bit product per piece, four quarter-rate multiplies, the walks took
// (a training step, us) 497 in place of 487 on 32 heads of 2048 x 128, 228 in place of 226.5 on 64 of 2048 x 64.
template <int D> struct Piece {
  uint32_t off, colb;
  int sn;
  __device__ __forceinline__ Piece(const Rows<D>& r, int64_t row_stride)
      : off(4u * (uint32_t)(r.row * (int)row_stride + r.col)), colb(4u * (uint32_t)r.col), sn((int)row_stride) {}
  __device__ __forceinline__ void load(f32x4 (&x)[2], const float* head, int t0, int N) const {
    t0 = min(t0, N - 1);
    const int last = min(N - 1 - t0, CH - 1);
    const char* chunk = reinterpret_cast<const char*>(head + (int64_t)t0 * sn);
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int first = min(16 * p, last);
      const uint32_t lim = 4u * (uint32_t)((last - first) * sn) + colb;
      x[p] = *reinterpret_cast<const f32x4*>(chunk + 4u * (uint32_t)(first * sn) + (size_t)min(off, lim));
    }
  }
};
// This lane's four columns of token 16*tb + i of a chunk, on their way out.
struct OutPiece {
  uint32_t off;
  int sn;
  __device__ __forceinline__ OutPiece(int64_t row_stride, int wave, int g, int i)
      : off(4u * (uint32_t)(i * (int)row_stride + 16 * wave + 4 * g)), sn((int)row_stride) {}
  __device__ __forceinline__ void store(float* head, int t, f32x4 x) const {   // t: uniform
    *reinterpret_cast<f32x4*>(reinterpret_cast<char*>(head + (int64_t)t * sn) + (size_t)off) = x;
  }
};

// Walks the chunks of [begin, end) upwards (downwards).  Whole chunks run as body(t0, true_type): with
// a condition in front of a load or a store the compiler has to assume that it may not have been
// issued, and then waits for everything outstanding, the last chunk's stores included, before it
// stages the next chunk.  Loads past the end are clamped to the last row.
template <typename Body> __device__ __forceinline__ void walk_forward(int begin, int end, Body body) {
  int t0 = begin;
  for (; t0 + CH <= end; t0 += CH) body(t0, std::true_type{});
  if (t0 < end) body(t0, std::false_type{});
}
template <typename Body> __device__ __forceinline__ void walk_backward(int begin, int end, Body body) {
  int t0 = begin + (end - begin - 1) / CH * CH;
  if (t0 + CH > end) {
    body(t0, std::false_type{});
    t0 -= CH;
  }
  for (; t0 >= begin; t0 -= CH) body(t0, std::true_type{});
}

// Carried sum as wave w holds it: tile 4*hh + x, register r, lane (g, i) is
//   by value column:    feature 64*hh + 16*g + 4*r + x, value   16*w + i   (kByValue)
//   by feature column:  value   64*hh + 16*g + 4*r + x, feature 16*w + i   (kByFeature)
template <int D, bool BY_VALUE>
__device__ __forceinline__ void add_sum(f32x4 (&s)[D / 16], const float* src, int wave, int g, int i) {
#pragma unroll
  for (int hh = 0; hh < D / 64; ++hh)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 64 * hh + 16 * g + 4 * r, col = 16 * wave + i;
      if constexpr (BY_VALUE) {
#pragma unroll
        for (int x = 0; x < 4; ++x) s[4 * hh + x][r] += src[(row + x) * D + col];
      } else {
        const f32x4 v = *reinterpret_cast<const f32x4*>(src + col * D + row);
#pragma unroll
        for (int x = 0; x < 4; ++x) s[4 * hh + x][r] += v[x];
      }
    }
}
template <int D, bool BY_VALUE>
__device__ __forceinline__ void put_sum(const f32x4 (&s)[D / 16], float* dst, int wave, int g, int i) {
#pragma unroll
  for (int hh = 0; hh < D / 64; ++hh)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 64 * hh + 16 * g + 4 * r, col = 16 * wave + i;
      if constexpr (BY_VALUE) {
#pragma unroll
        for (int x = 0; x < 4; ++x) dst[(row + x) * D + col] = s[4 * hh + x][r];
      } else {
        *reinterpret_cast<f32x4*>(dst + col * D + row) =
            f32x4{s[4 * hh][r], s[4 * hh + 1][r], s[4 * hh + 2][r], s[4 * hh + 3][r]};
      }
    }
}
template <int D> __device__ __forceinline__ void clear(f32x4 (&s)[D / 16]) {
#pragma unroll
  for (int t = 0; t < D / 16; ++t) s[t] = kZeroF4;
}

// s += sum over the chunk's tokens of (row of `tall`)^T (x) `col`: col[ub][r] is this lane's column of
// token 16*ub + 4*g + r.
template <int D>
__device__ __forceinline__ void add_outer(f32x4 (&s)[D / 16], const float* tall, const float (&col)[2][4], int g, int i) {
#pragma unroll
  for (int ub = 0; ub < 2; ++ub)
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int hh = 0; hh < D / 64; ++hh) {
        const f32x4 x = lds4(tall + (16 * ub + 4 * g + r) * kF32Row<D> + 64 * hh + 4 * i);
#pragma unroll
        for (int j = 0; j < 4; ++j) s[4 * hh + j] = mfma_f32(x[j], col[ub][r], s[4 * hh + j]);
      }
}
// out[tb] += s^T applied to rows 16*tb + i of `rows`: column 16*w + row of the result, one token a lane
template <int D>
__device__ __forceinline__ void read_out(f32x4 (&out)[2], const f32x4 (&s)[D / 16], const float* rows, int g, int i) {
#pragma unroll
  for (int hh = 0; hh < D / 64; ++hh)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int off = i * kF32Row<D> + 64 * hh + 16 * g + 4 * r;
      const f32x4 x0 = lds4(rows + off), x1 = lds4(rows + 16 * kF32Row<D> + off);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        out[0] = mfma_f32(s[4 * hh + j][r], x0[j], out[0]);
        out[1] = mfma_f32(s[4 * hh + j][r], x1[j], out[1]);
      }
    }
}
// this lane's column (16*w + i) of the chunk's tokens, in add_outer's order
template <int D>
__device__ __forceinline__ void column(float (&c)[2][4], const float* tile, int wave, int g, int i) {
#pragma unroll
  for (int ub = 0; ub < 2; ++ub)
#pragma unroll
    for (int r = 0; r < 4; ++r) c[ub][r] = tile[(16 * ub + 4 * g + r) * kF32Row<D> + 16 * wave + i];
}
__device__ __forceinline__ float sum8(const float (&c)[2][4]) {
  return sum_over_groups(((c[0][0] + c[0][1]) + (c[0][2] + c[0][3])) + ((c[1][0] + c[1][1]) + (c[1][2] + c[1][3])));
}

// ---- sum of phi(k) (x) v and phi(k) over every segment ------------------------------------------
struct StateArgs {
  TensorView k, v;
  float* sums;        // [heads][nseg][d*d + d]
  int H0, H1, N, phi;
  int seg_len, nseg;  // tokens per segment (a multiple of CH), segments per head
  int per_head;       // segments summed: all of them, or (causal) all but the last
};
template <int D>
__global__ __launch_bounds__(kLinThreads<D>, 2) void linear_f32_state_kernel(StateArgs a) {
  constexpr int TR = kF32Row<D>;
  __shared__ __attribute__((aligned(16))) float fk[CH * TR];
  __shared__ __attribute__((aligned(16))) float vv[CH * TR];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, i = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int seg = blockIdx.x % a.per_head, head = blockIdx.x / a.per_head;
  const int b = head / a.H1, h = a.H0 + head % a.H1;
  const float* kp = reinterpret_cast<const float*>(a.k.base) + b * a.k.sb + h * a.k.sh;
  const float* vp = reinterpret_cast<const float*>(a.v.base) + b * a.v.sb + h * a.v.sh;
  const int begin = seg * a.seg_len, end = min(a.N, begin + a.seg_len);
  const Rows<D> st(tid);
  f32x4 s[D / 16], kr[2], vr[2];
  clear<D>(s);
  float z = 0.f;
  const Piece<D> pk(st, a.k.sn), pv(st, a.v.sn);
  pk.load(kr, kp, begin, a.N);
  pv.load(vr, vp, begin, a.N);
  for (int t0 = begin; t0 < end; t0 += CH) {
    lds_barrier();
    st.store_mapped(fk, kr, t0, a.N, a.phi);
    st.store(vv, vr, t0, a.N);
    if (t0 + CH < end) {
      pk.load(kr, kp, t0 + CH, a.N);
      pv.load(vr, vp, t0 + CH, a.N);
    }
    lds_barrier();
    float vc[2][4], kc[2][4];
    column<D>(vc, vv, wave, g, i);
    add_outer<D>(s, fk, vc, g, i);
    column<D>(kc, fk, wave, g, i);
    z += sum8(kc);
  }
  float* dst = a.sums + ((int64_t)head * a.nseg + seg) * kLinState<D>;
  put_sum<D, true>(s, dst, wave, g, i);
  if (g == 0) dst[D * D + 16 * wave + i] = z;
}

// A thread owns four neighbouring floats of every slot and has sixteen slots in flight, one trip to memory for most
// calls (one float and eight slots: 2 x 16 x 9000 tokens, bf16 backward, 137.5 -> 134.3 us; 64 heads x 4096 114.7 -> 113.2).
// Every head's sums become what each segment starts from
// (mode 0: sums of the segments before; 1: of the segments behind; 2: slot 0 receives the total).
__global__ __launch_bounds__(64) void segment_scan_kernel(float* sums, int nseg, int floats, int mode) {
  const int x = 4 * (blockIdx.x * 64 + threadIdx.x);
  if (x >= floats) return;
  float* p = sums + (int64_t)blockIdx.y * nseg * floats + x;
  constexpr int G = 16;   // loads in flight
  f32x4 run = kZeroF4;
  for (int j0 = 0; j0 < nseg; j0 += G) {
    f32x4 v[G];
#pragma unroll
    for (int j = 0; j < G; ++j) {
      const int k = min(j0 + j, nseg - 1);
      v[j] = *reinterpret_cast<const f32x4*>(p + (int64_t)(mode == 1 ? nseg - 1 - k : k) * floats);
    }
#pragma unroll
    for (int j = 0; j < G; ++j)
      if (j0 + j < nseg) {
        if (mode != 2) *reinterpret_cast<f32x4*>(p + (int64_t)(mode == 1 ? nseg - 1 - j0 - j : j0 + j) * floats) = run;
        run += v[j];
      }
  }
  if (mode == 2) *reinterpret_cast<f32x4*>(p) = run;
}

// The slots [first, last) a segment's walk adds up.
__device__ __forceinline__ void slots_before(bool causal, int seg, int nseg, int& first, int& last) {
  if (nseg > kSumInPlace) { first = causal ? seg : 0; last = first + 1; }
  else { first = 0; last = causal ? seg : nseg; }
}
__device__ __forceinline__ void slots_behind(bool causal, int seg, int nseg, int& first, int& last) {
  if (nseg > kSumInPlace) { first = causal ? seg : 0; last = first + 1; }
  else { first = causal ? seg + 1 : 0; last = nseg; }
}

// ---- forward ---------------------------------------------------------------------------------
template <int D> struct F32FwdSmem {
  float fq[CH * kF32Row<D>], fk[CH * kF32Row<D>], vv[CH * kF32Row<D>];
  float p[CH * PR];   // masked products [query][key]
  float z[D];
};
template <int D, bool CAUSAL>
__device__ __forceinline__ void linear_f32(const AttnArgs& a, int block, unsigned char* smem_raw) {
  constexpr int TR = kF32Row<D>;
  F32FwdSmem<D>& sm = *reinterpret_cast<F32FwdSmem<D>*>(smem_raw);
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, i = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = a.N, H1 = a.H - a.H0;
  const int seg = block % a.f32_nseg, head = block / a.f32_nseg;
  const int b = head / H1, h = a.H0 + head % H1;
  const float* qp = reinterpret_cast<const float*>(a.q.base) + b * a.q.sb + h * a.q.sh;
  const float* kp = reinterpret_cast<const float*>(a.k.base) + b * a.k.sb + h * a.k.sh;
  const float* vp = reinterpret_cast<const float*>(a.v.base) + b * a.v.sb + h * a.v.sh;
  float* op = reinterpret_cast<float*>(a.out) + b * a.osb + h * a.osh;
  const int begin = seg * a.f32_seg_len, end = min(N, begin + a.f32_seg_len);
  const Rows<D> st(tid);
  const Piece<D> pq(st, a.q.sn), pk(st, a.k.sn), pv(st, a.v.sn);
  const OutPiece oo(a.osn, wave, g, i);
  f32x4 s[D / 16], qr[2], kr[2], vr[2];
  pq.load(qr, qp, begin, N);
  if (CAUSAL) {
    pk.load(kr, kp, begin, N);
    pv.load(vr, vp, begin, N);
  }
  clear<D>(s);
  {
    int first, last;
    slots_before(CAUSAL, seg, a.f32_nseg, first, last);
    float z = 0.f;
    for (int j = first; j < last; ++j) {
      const float* src = a.ws_states + ((int64_t)head * a.f32_nseg + j) * kLinState<D>;
      add_sum<D, true>(s, src, wave, g, i);
      if (tid < D) z += src[D * D + tid];
    }
    if (tid < D) sm.z[tid] = z;
  }
  // STEADY: a whole chunk, whose loads and stores carry no condition (see walk_forward)
  walk_forward(begin, end, [&](int t0, auto steady) {
    constexpr bool STEADY = decltype(steady)::value;
    lds_barrier();   // the chunk before is consumed
    st.store_mapped(sm.fq, qr, t0, N, a.phi);
    if (CAUSAL) {
      st.store_mapped(sm.fk, kr, t0, N, a.phi);
      st.store(sm.vv, vr, t0, N);
    }
    if (STEADY || t0 + CH < end) {
      pq.load(qr, qp, t0 + CH, N);
      if (CAUSAL) {
        pk.load(kr, kp, t0 + CH, N);
        pv.load(vr, vp, t0 + CH, N);
      }
    }
    lds_barrier();
    if (CAUSAL && wave < 3) {   // masked products, 16 queries x 16 keys a wave
      const int tb = wave > 0, ub = wave > 1;
      f32x4 p = rows_product_lds<D>(sm.fk + (16 * ub + i) * TR + 4 * g, sm.fq + (16 * tb + i) * TR + 4 * g);
#pragma unroll
      for (int r = 0; r < 4; ++r) p[r] = (tb != ub || 4 * g + r <= i) ? p[r] : 0.f;
      *reinterpret_cast<f32x4*>(sm.p + (16 * tb + i) * PR + 16 * ub + 4 * g) = p;
    }
    f32x4 num[2] = {kZeroF4, kZeroF4};
    read_out<D>(num, s, sm.fq, g, i);
    float den[2] = {0.f, 0.f};
#pragma unroll
    for (int c = 0; c < D; c += 16) {
      const f32x4 z = lds4(sm.z + c + 4 * g);
#pragma unroll
      for (int tb = 0; tb < 2; ++tb) {
        const f32x4 f = lds4(sm.fq + (16 * tb + i) * TR + c + 4 * g);
#pragma unroll
        for (int j = 0; j < 4; ++j) den[tb] = fmaf(f[j], z[j], den[tb]);
      }
    }
    float vc[2][4];
    if (CAUSAL) {
      lds_barrier();   // products visible
      column<D>(vc, sm.vv, wave, g, i);
#pragma unroll
      for (int tb = 0; tb < 2; ++tb)
#pragma unroll
        for (int ub = 0; ub <= tb; ++ub) {
          const f32x4 p = lds4(sm.p + (16 * tb + i) * PR + 16 * ub + 4 * g);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            num[tb] = mfma_f32(vc[ub][r], p[r], num[tb]);
            den[tb] += p[r];
          }
        }
    }
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) {
      // the reciprocal of den without its power of two, 2^e: below 2.9e-39 den has none (features of small
      // products).  Eight divisions a lane instead: 72.4 against 69.9 us on 64 heads x 2048 x 64.
      const float dt = sum_over_groups(den[tb]) + a.eps;
      const int e = __builtin_amdgcn_frexp_expf(dt) - 1;   // -1 for 0 and infinity, whose reciprocals stay theirs
      const float inv = 1.f / __builtin_amdgcn_ldexpf(dt, -e);
      f32x4 o;
#pragma unroll
      for (int j = 0; j < 4; ++j) o[j] = __builtin_amdgcn_ldexpf(num[tb][j] * inv, -e);
      const int n = t0 + 16 * tb + i;
      if (STEADY || n < N)
        oo.store(op, t0 + 16 * tb, o);
    }
    if (CAUSAL) {
      add_outer<D>(s, sm.fk, vc, g, i);
      float kc[2][4];
      column<D>(kc, sm.fk, wave, g, i);
      const float dz = sum8(kc);
      if (g == 0) sm.z[16 * wave + i] += dz;   // last read in front of the barrier above
    }
  });
  if (CAUSAL && a.final_state && end == N) {   // what a decode step continues from
    float* fs = a.final_state + (int64_t)head * kLinState<D>;
    put_sum<D, true>(s, fs, wave, g, i);
    if (g == 0) fs[D * D + 16 * wave + i] = sm.z[16 * wave + i];
  }
}

// ---- backward, forward walk: dq, (den, c), and the segment's sums (B, Y) --------------------------
// The products with dO come before the division by den, which is known last.  So that none of them leaves the
// range of a float where dO / den is inside it, a row of dO enters as its power of two, 2^e, times the rest:
// products with the rest are as large as den and A are, and 2^e / den is applied to them (a training step of
// 4 x (3 + 13 heads) x 2048 x 64: 293.9 us without, 296.1 with).
template <int D> struct F32BwdSmem {
  float fq[CH * kF32Row<D>], fk[CH * kF32Row<D>], vv[CH * kF32Row<D>], dd[CH * kF32Row<D>];
  float p[CH * PR], w[CH * PR];      // masked phi(q).phi(k) and dO.v products
  float z[D];                        // Z (dq walk) or Y (dk, dv walk)
  float red[2][D / 16][CH];          // per-wave parts of phi(q).r and phi(q).Z; c of the chunk
  int exps[CH];                      // the powers of two taken out of dO's rows (dq walk)
};
template <int D, bool CAUSAL>
__device__ __forceinline__ void linear_bwd_q_f32(const BwdArgs& a, int block, unsigned char* smem_raw) {
  constexpr int TR = kF32Row<D>, NW = D / 16;
  F32BwdSmem<D>& sm = *reinterpret_cast<F32BwdSmem<D>*>(smem_raw);
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, i = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = a.N, H1 = a.H - a.H0;
  const int seg = block % a.f32_nseg, head = block / a.f32_nseg;
  const int b = head / H1, h = a.H0 + head % H1;
  const float* qp = reinterpret_cast<const float*>(a.q.base) + b * a.q.sb + h * a.q.sh;
  const float* kp = reinterpret_cast<const float*>(a.k.base) + b * a.k.sb + h * a.k.sh;
  const float* vp = reinterpret_cast<const float*>(a.v.base) + b * a.v.sb + h * a.v.sh;
  const float* dp = reinterpret_cast<const float*>(a.dout.base) + b * a.dout.sb + h * a.dout.sh;
  float* dq = reinterpret_cast<float*>(a.dq) + b * a.q.sb + h * a.q.sh;
  float* ws = a.ws + ((int64_t)b * a.H + h) * N * 2;
  const int begin = seg * a.f32_seg_len, end = min(N, begin + a.f32_seg_len);
  const Rows<D> st(tid);
  const Piece<D> pq(st, a.q.sn), pk(st, a.k.sn), pv(st, a.v.sn), pd(st, a.dout.sn);
  const OutPiece oq(a.q.sn, wave, g, i);
  f32x4 qr[2], kr[2], vr[2], dr[2];
  auto load = [&](int t0) {
    pq.load(qr, qp, t0, N);
    pd.load(dr, dp, t0, N);
    if (CAUSAL) {
      pk.load(kr, kp, t0, N);
      pv.load(vr, vp, t0, N);
    }
  };
  load(begin);
  f32x4 s[D / 16], bs[D / 16];   // A and this segment's B, both by feature column
  clear<D>(s);
  clear<D>(bs);
  float y = 0.f;
  {
    int first, last;
    slots_before(CAUSAL, seg, a.f32_nseg, first, last);
    float z = 0.f;
    for (int j = first; j < last; ++j) {
      const float* src = a.ws_state + ((int64_t)head * a.f32_nseg + j) * kLinState<D>;
      add_sum<D, false>(s, src, wave, g, i);
      if (tid < D) z += src[D * D + tid];
    }
    if (tid < D) sm.z[tid] = z;
  }
  walk_forward(begin, end, [&](int t0, auto steady) {
    constexpr bool STEADY = decltype(steady)::value;
    lds_barrier();
    st.store_mapped(sm.fq, qr, t0, N, a.phi);
    st.store_normalised(sm.dd, dr, sm.exps, t0, N);
    if (CAUSAL) {
      st.store_mapped(sm.fk, kr, t0, N, a.phi);
      st.store(sm.vv, vr, t0, N);
    }
    if (STEADY || t0 + CH < end) load(t0 + CH);
    lds_barrier();
    if (CAUSAL) {
      // phi(q_t).phi(k_u) and dO_t.v_u, u <= t: [query][key]
      for (int x = wave; x < 6; x += NW) {
        const int t = x % 3, tb = t > 0, ub = t > 1;
        const float* keys = x < 3 ? sm.fk : sm.vv;
        const float* rows = x < 3 ? sm.fq : sm.dd;
        f32x4 p = rows_product_lds<D>(keys + (16 * ub + i) * TR + 4 * g, rows + (16 * tb + i) * TR + 4 * g);
#pragma unroll
        for (int r = 0; r < 4; ++r) p[r] = (tb != ub || 4 * g + r <= i) ? p[r] : 0.f;
        *reinterpret_cast<f32x4*>((x < 3 ? sm.p : sm.w) + (16 * tb + i) * PR + 16 * ub + 4 * g) = p;
      }
    }
    // r_t = A dO_t (the division by den follows): features 16w + 4g + j, token 16 tb + i
    f32x4 rv[2] = {kZeroF4, kZeroF4};
    read_out<D>(rv, s, sm.dd, g, i);
    const f32x4 zc = lds4(sm.z + 16 * wave + 4 * g);
    f32x4 qc[2];
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) {
      qc[tb] = lds4(sm.fq + (16 * tb + i) * TR + 16 * wave + 4 * g);
      float qrv = 0.f, qz = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        qrv = fmaf(qc[tb][j], rv[tb][j], qrv);
        qz = fmaf(qc[tb][j], zc[j], qz);
      }
      qrv = sum_over_groups(qrv);
      qz = sum_over_groups(qz);
      if (g == 0) {
        sm.red[0][wave][16 * tb + i] = qrv;
        sm.red[1][wave][16 * tb + i] = qz;
      }
    }
    lds_barrier();   // products and parts visible
    float kc[2][4];
    if (CAUSAL) column<D>(kc, sm.fk, wave, g, i);
    float inv[2], cv[2];   // 2^e / den and c
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) {
      const int n = t0 + 16 * tb + i;
      float qrv = 0.f, qz = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        qrv += sm.red[0][w][16 * tb + i];
        qz += sm.red[1][w][16 * tb + i];
      }
      f32x4 wv[2];
      if (CAUSAL) {
        float ps = 0.f, pw = 0.f;
#pragma unroll
        for (int ub = 0; ub <= tb; ++ub) {
          const f32x4 p = lds4(sm.p + (16 * tb + i) * PR + 16 * ub + 4 * g);
          wv[ub] = lds4(sm.w + (16 * tb + i) * PR + 16 * ub + 4 * g);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            ps += p[r];
            pw = fmaf(p[r], wv[ub][r], pw);
          }
        }
        qz += sum_over_groups(ps);
        qrv += sum_over_groups(pw);
      }
      const float den = STEADY || n < N ? qz + a.eps : 1.f;   // rows past the end: dO is zero
      inv[tb] = __builtin_amdgcn_ldexpf(1.f, sm.exps[16 * tb + i]) / den;
      cv[tb] = qrv / den * inv[tb];
      if (STEADY || n < N)   // every wave and lane group has the same values for the token
        *reinterpret_cast<float2*>(ws + 2 * (int64_t)n) = make_float2(den, cv[tb]);
      f32x4 acc;
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j] = rv[tb][j] * inv[tb] - cv[tb] * zc[j];
      if (CAUSAL) {
#pragma unroll
        for (int ub = 0; ub <= tb; ++ub)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float w = (tb != ub || 4 * g + r <= i) ? fmaf(wv[ub][r], inv[tb], -cv[tb]) : 0.f;
            acc = mfma_f32(kc[ub][r], w, acc);
          }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j] *= feature_map_slope(qc[tb][j], a.phi);
      if (STEADY || n < N) {
        oq.store(dq, t0 + 16 * tb, acc);
      }
    }
    // B += phi(q)^T (x) dO / den, Y += c phi(q); a token's 2^e / den and c sit in the lane that owns it
    float qcol[2][4];
    column<D>(qcol, sm.fq, wave, g, i);
#pragma unroll
    for (int ub = 0; ub < 2; ++ub)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        y = fmaf(__shfl(cv[ub], 4 * g + r, 64), qcol[ub][r], y);
        qcol[ub][r] *= __shfl(inv[ub], 4 * g + r, 64);
      }
    add_outer<D>(bs, sm.dd, qcol, g, i);
    if (CAUSAL) {
      add_outer<D>(s, sm.vv, kc, g, i);
      const float dz = sum8(kc);
      if (g == 0) sm.z[16 * wave + i] += dz;   // read by this wave alone
    }
  });
  if (CAUSAL && seg == 0) return;   // nothing lies in front of a head's first segment
  float* dst = a.ws_state + ((int64_t)a.B * H1 * a.f32_nseg + (int64_t)head * a.f32_nseg + seg) * kLinState<D>;
  put_sum<D, false>(bs, dst, wave, g, i);
  y = sum_over_groups(y);
  if (g == 0) dst[D * D + 16 * wave + i] = y;
}

// ---- backward, reverse walk: dk and dv -----------------------------------------------------------
// B is an operand by feature column (dk) and by value column (dv).  Accumulated in both orders it took a fifth of the
// walk's matrix instructions twice, and twice the loads of the sums it starts from; now the waves keep it by feature column and
// leave a copy, turned, in LDS.  A training step, us, before and after: 4 x (3 + 13) x 2048 x 64 266.5 and 260.0, 4 x 16 x
// 1024 x 128 540 and 517.
template <int D> struct F32BwdKvSmem : F32BwdSmem<D> {
  float b[D * kF32Row<D>];           // [value][feature], row v rotated by 16 * (v / 16) floats: writes and reads miss each other's banks
};
template <int D> __device__ __forceinline__ int turned(int value, int feature) {
  return value * kF32Row<D> + (feature + (value & ~15)) % D;
}
template <int D, bool CAUSAL>
__device__ __forceinline__ void linear_bwd_kv_f32(const BwdArgs& a, int block, unsigned char* smem_raw) {
  constexpr int TR = kF32Row<D>, NW = D / 16;
  F32BwdKvSmem<D>& sm = *reinterpret_cast<F32BwdKvSmem<D>*>(smem_raw);
  float* cvec = &sm.red[0][0][0];   // c of the chunk's tokens
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, i = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = a.N, H1 = a.H - a.H0;
  const int seg = block % a.f32_nseg, head = block / a.f32_nseg;
  const int b = head / H1, h = a.H0 + head % H1;
  const float* qp = reinterpret_cast<const float*>(a.q.base) + b * a.q.sb + h * a.q.sh;
  const float* kp = reinterpret_cast<const float*>(a.k.base) + b * a.k.sb + h * a.k.sh;
  const float* vp = reinterpret_cast<const float*>(a.v.base) + b * a.v.sb + h * a.v.sh;
  const float* dp = reinterpret_cast<const float*>(a.dout.base) + b * a.dout.sb + h * a.dout.sh;
  float* dk = reinterpret_cast<float*>(a.dk) + b * a.k.sb + h * a.k.sh;
  float* dv = reinterpret_cast<float*>(a.dv) + b * a.v.sb + h * a.v.sh;
  const float* ws = a.ws + ((int64_t)b * a.H + h) * N * 2;
  const int begin = seg * a.f32_seg_len, end = min(N, begin + a.f32_seg_len);
  const Rows<D> st(tid);
  const Piece<D> pq(st, a.q.sn), pk(st, a.k.sn), pv(st, a.v.sn), pd(st, a.dout.sn);
  const OutPiece ok(a.k.sn, wave, g, i), ov(a.v.sn, wave, g, i);
  f32x4 qr[2], kr[2], vr[2], dr[2];
  float den[2], cr = 0.f;
  auto load = [&](int t0) {
    pk.load(kr, kp, t0, N);
    pv.load(vr, vp, t0, N);
    if (CAUSAL) {
      pq.load(qr, qp, t0, N);
      pd.load(dr, dp, t0, N);
#pragma unroll
      for (int p = 0; p < 2; ++p) den[p] = ws[2 * (int64_t)min(t0 + st.row + 16 * p, N - 1)];
      if (tid < CH) cr = t0 + tid < N ? ws[2 * (int64_t)(t0 + tid) + 1] : 0.f;
    }
  };
  f32x4 b1[D / 16];   // B by feature column
  clear<D>(b1);
  const int last_chunk = begin + (end - begin - 1) / CH * CH;
  load(last_chunk);
  {
    const float* sums = a.ws_state + ((int64_t)a.B * H1 + head) * a.f32_nseg * kLinState<D>;
    int first, last;
    slots_behind(CAUSAL, seg, a.f32_nseg, first, last);
    float yz = 0.f;
    for (int j = first; j < last; ++j) {
      const float* src = sums + (int64_t)j * kLinState<D>;
      add_sum<D, false>(b1, src, wave, g, i);
      if (tid < D) yz += src[D * D + tid];
    }
    if (tid < D) sm.z[tid] = yz;
  }
  auto copy_b = [&]() {
#pragma unroll
    for (int hh = 0; hh < D / 64; ++hh)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int x = 0; x < 4; ++x) sm.b[turned<D>(64 * hh + 16 * g + 4 * r + x, 16 * wave + i)] = b1[4 * hh + x][r];
  };
  copy_b();
  walk_backward(begin, end, [&](int t0, auto steady) {
    constexpr bool STEADY = decltype(steady)::value;
    lds_barrier();
    st.store_mapped(sm.fk, kr, t0, N, a.phi);
    st.store(sm.vv, vr, t0, N);
    if (CAUSAL) {
      st.store_mapped(sm.fq, qr, t0, N, a.phi);
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int j = 0; j < 4; ++j) dr[p][j] /= den[p];   // g = dO / den
      st.store(sm.dd, dr, t0, N);
      if (tid < CH) cvec[tid] = cr;
    }
    if (STEADY || t0 - CH >= begin) load(max(t0 - CH, begin));
    lds_barrier();
    if (CAUSAL) {
      // phi(q_t).phi(k_u) and g_t.v_u - c_t, t >= u: [key][query]
      for (int x = wave; x < 6; x += NW) {
        const int t = x % 3, ub = t > 1, tb = t > 0;
        const float* rows = x < 3 ? sm.fq : sm.dd;
        const float* keys = x < 3 ? sm.fk : sm.vv;
        f32x4 p = rows_product_lds<D>(rows + (16 * tb + i) * TR + 4 * g, keys + (16 * ub + i) * TR + 4 * g);
        if (x >= 3) p -= lds4(cvec + 16 * tb + 4 * g);
#pragma unroll
        for (int r = 0; r < 4; ++r) p[r] = (tb != ub || 4 * g + r >= i) ? p[r] : 0.f;
        *reinterpret_cast<f32x4*>((x < 3 ? sm.p : sm.w) + (16 * ub + i) * PR + 16 * tb + 4 * g) = p;
      }
    }
    const f32x4 yc = lds4(sm.z + 16 * wave + 4 * g);
    f32x4 dka[2], dva[2];
#pragma unroll
    for (int ub = 0; ub < 2; ++ub) { dka[ub] = -yc; dva[ub] = kZeroF4; }
    read_out<D>(dka, b1, sm.vv, g, i);
#pragma unroll
    for (int hh = 0; hh < D / 64; ++hh)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int f0 = 64 * hh + 16 * g + 4 * r;
        const f32x4 s = lds4(sm.b + turned<D>(16 * wave + i, f0));
        const f32x4 x0 = lds4(sm.fk + i * TR + f0), x1 = lds4(sm.fk + (16 + i) * TR + f0);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          dva[0] = mfma_f32(s[j], x0[j], dva[0]);
          dva[1] = mfma_f32(s[j], x1[j], dva[1]);
        }
      }
    float qcol[2][4], gcol[2][4];
    if (CAUSAL) {
      lds_barrier();   // products visible
      column<D>(qcol, sm.fq, wave, g, i);
      column<D>(gcol, sm.dd, wave, g, i);
#pragma unroll
      for (int ub = 0; ub < 2; ++ub)
#pragma unroll
        for (int tb = ub; tb < 2; ++tb) {
          const f32x4 w = lds4(sm.w + (16 * ub + i) * PR + 16 * tb + 4 * g);
          const f32x4 p = lds4(sm.p + (16 * ub + i) * PR + 16 * tb + 4 * g);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            dka[ub] = mfma_f32(qcol[tb][r], w[r], dka[ub]);
            dva[ub] = mfma_f32(gcol[tb][r], p[r], dva[ub]);
          }
        }
    }
#pragma unroll
    for (int ub = 0; ub < 2; ++ub) {
      const int n = t0 + 16 * ub + i;
      const f32x4 kc = lds4(sm.fk + (16 * ub + i) * TR + 16 * wave + 4 * g);
#pragma unroll
      for (int j = 0; j < 4; ++j) dka[ub][j] *= feature_map_slope(kc[j], a.phi);
      if (STEADY || n < N) {
        ok.store(dk, t0 + 16 * ub, dka[ub]);
        ov.store(dv, t0 + 16 * ub, dva[ub]);
      }
    }
    if (CAUSAL) {
      add_outer<D>(b1, sm.dd, qcol, g, i);
      copy_b();   // last read in front of the barrier above
      float dy = 0.f;
#pragma unroll
      for (int tb = 0; tb < 2; ++tb) {
        const f32x4 c = lds4(cvec + 16 * tb + 4 * g);
#pragma unroll
        for (int r = 0; r < 4; ++r) dy = fmaf(c[r], qcol[tb][r], dy);
      }
      dy = sum_over_groups(dy);
      if (g == 0) sm.z[16 * wave + i] += dy;   // read by this wave alone
    }
  });
}

template <int D>
hipError_t launch_states(const TensorView& k, const TensorView& v, float* sums, int B, int H0, int H1, int N,
                         int phi, int seg_len, int nseg, bool causal, hipStream_t s) {
  const int per_head = causal ? nseg - 1 : nseg;
  if (per_head <= 0) return hipSuccess;
  const StateArgs sa{k, v, sums, H0, H1, N, phi, seg_len, nseg, per_head};
  linear_f32_state_kernel<D><<<dim3(B * H1 * per_head), dim3(kLinThreads<D>), 0, s>>>(sa);
  return hipGetLastError();
}
hipError_t launch_scan(float* sums, int heads, int nseg, int floats, int mode, hipStream_t s) {
  return nseg <= kSumInPlace ? hipSuccess : launch_segment_scan(sums, heads, nseg, floats, mode, s);
}
// A walk, and at d = 64 behind it in the same launch (from the next multiple of 8 on, so that the XCDs keep
// their runs) the `band` workgroups of the windowed heads that go with it.  Same bits as apart.
// Measured (a training step of 4 x (3 + 13 heads) x 2048 x 64, window 128, us): 319 apart, 294 together; read-out
// 39 + 22 -> 58, dq 57 + 45 -> 98, dk and dv 64 + 35 -> 99, and three launches less.  The last keeps the windowed
// heads' 194 registers; the walk's own LDS, 63 KB with the turned copy of B (147 at d = 128), lets no more than two workgroups
// (one) share a compute unit either.
enum Walk { kReadOut, kQWalk, kKvWalk };
template <int D, bool CAUSAL, int WALK, typename Args>
__global__ __launch_bounds__(kLinThreads<D>, 2) void linear_f32_walk_kernel(Args a, int linear, int band) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  const int block = blockIdx.x, first = (linear + 7) & ~7;
  if (block < linear) {
    if constexpr (WALK == kReadOut) linear_f32<D, CAUSAL>(a, block, smem_raw);
    else if constexpr (WALK == kQWalk) linear_bwd_q_f32<D, CAUSAL>(a, block, smem_raw);
    else linear_bwd_kv_f32<D, CAUSAL>(a, block, smem_raw);
  } else if constexpr (D == 64) {
    static_assert(kLinThreads<64> == kF32BandThreads, "one block size for both kinds of workgroup");
    if (block < first || band == 0) return;
    if constexpr (WALK == kReadOut) windowed_f32<D, 4>(a, block - first, smem_raw);
    else if constexpr (WALK == kQWalk) windowed_bwd_q_f32<D, 4>(a, block - first, smem_raw);
    else windowed_bwd_kv_f32<D, 4>(a, block - first, smem_raw);
  }
}
template <int D, int WALK, typename A>
hipError_t launch_walk(const A& a, int linear, int band, size_t smem, hipStream_t s) {
  if (band > 0 && smem < sizeof(F32WinSmem<D>)) smem = sizeof(F32WinSmem<D>);
  auto launch = [&](auto kern) {
    const hipError_t e = allow_lds(kern, smem);
    if (e != hipSuccess) return e;
    kern<<<dim3(band > 0 ? ((linear + 7) & ~7) + band : linear), dim3(kLinThreads<D>), smem, s>>>(a, linear, band);
    return hipGetLastError();
  };
  return a.causal ? launch(linear_f32_walk_kernel<D, true, WALK, A>) : launch(linear_f32_walk_kernel<D, false, WALK, A>);
}
// workgroups of the windowed heads that ride along
template <int D, typename A> int band_blocks(const A& a, bool with_windowed) {
  return with_windowed ? (a.N + 63) / 64 * a.H0 * a.B : 0;
}

template <int D> hipError_t forward(const AttnArgs& a, bool with_windowed, hipStream_t s) {
  const int H1 = a.H - a.H0, heads = a.B * H1, blocks = heads * a.f32_nseg;
  hipError_t e = launch_states<D>(a.k, a.v, a.ws_states, a.B, a.H0, H1, a.N, a.phi, a.f32_seg_len, a.f32_nseg, a.causal, s);
  if (e == hipSuccess) e = launch_scan(a.ws_states, heads, a.f32_nseg, kLinState<D>, a.causal ? 0 : 2, s);
  if (e != hipSuccess) return e;
  return launch_walk<D, kReadOut>(a, blocks, band_blocks<D>(a, with_windowed), sizeof(F32FwdSmem<D>), s);
}
template <int D> hipError_t backward(const BwdArgs& a, bool with_windowed, hipStream_t s) {
  const int H1 = a.H - a.H0, heads = a.B * H1, blocks = heads * a.f32_nseg;
  const int band = band_blocks<D>(a, with_windowed);
  float* bsums = a.ws_state + (int64_t)heads * a.f32_nseg * kLinState<D>;
  hipError_t e = launch_states<D>(a.k, a.v, a.ws_state, a.B, a.H0, H1, a.N, a.phi, a.f32_seg_len, a.f32_nseg, a.causal, s);
  if (e == hipSuccess) e = launch_scan(a.ws_state, heads, a.f32_nseg, kLinState<D>, a.causal ? 0 : 2, s);
  if (e == hipSuccess)
    e = launch_walk<D, kQWalk>(a, blocks, band, sizeof(F32BwdSmem<D>), s);
  if (e == hipSuccess) e = launch_scan(bsums, heads, a.f32_nseg, kLinState<D>, a.causal ? 1 : 2, s);
  if (e == hipSuccess)
    e = launch_walk<D, kKvWalk>(a, blocks, band, sizeof(F32BwdKvSmem<D>), s);
  return e;
}

}  // namespace

// A causal call takes as long as the compute unit with the most chunks to walk, one after the other, so a cut is priced
// by that number: 8 segments of 8 chunks a head are 2 x 8 on 256 units and 64 heads, 11 of 6 are 3 x 6 on some.  Two
// workgroups a unit hide each other's barriers nearly as well as three (1.1: the matrix units bind either way), one
// alone does not (1.7), and four are a second round (not considered).  Beyond kSumInPlace segments the sums are scanned
// by launches of their own, which cost as much as three chunks on a full unit, half as many on one that runs fast
// because it is alone; between equals the fewer segments.  Over all keys, where a walk adds up all of a head's sums
// and chunks are cheap, as many segments as give three workgroups a unit.  Measured (a training step, us; three
// workgroups a unit, this rule): 4 x (3 + 13) x 2048 x 64 291.3 -> 269.6 (13, 8 segments), without windowed heads
// 258.2 -> 228.5 (11, 8); elsewhere the same to 1 %.  (Then the dk/dv walk had room for three a unit as well; it has for
// two now, and 109 random backward calls, over all keys among them, are none of them slower by more than 1 %.)
Segments f32_segments(int64_t heads, int N, int d, bool causal, uint64_t bytes, int sums) {
  Segments f{N, 1};
  if (heads <= 0 || N <= 0) return f;
  const int64_t chunks = (N + CH - 1) / CH, cus = device_compute_units();
  const uint64_t room = bytes / ((uint64_t)heads * sums * ((uint64_t)d * d + d) * sizeof(float));
  int64_t most = std::min(std::min((int64_t)kMaxSegments, chunks / 4), 3 * cus / heads);
  if ((uint64_t)most > room) most = (int64_t)room;
  double best = 0.;
  for (int64_t n = causal ? 1 : std::max((int64_t)1, most); n <= most; ++n) {
    const int64_t len = (chunks + n - 1) / n, count = (chunks + len - 1) / len, per = (heads * count + cus - 1) / cus;
    const double cost = per * len * (per == 1 ? 1.7 : per == 2 ? 1.1 : 1.) + (count <= kSumInPlace ? 0. : per == 1 ? 1.5 : 3.);
    if (best == 0. || cost < best) {
      best = cost;
      f.count = (int)count;
      f.len = count > 1 ? (int)len * CH : N;
    }
  }
  return f;
}

hipError_t launch_segment_scan(float* sums, int heads, int nseg, int floats, int mode, hipStream_t s) {
  segment_scan_kernel<<<dim3((floats / 4 + 63) / 64, heads), dim3(64), 0, s>>>(sums, nseg, floats, mode);
  return hipGetLastError();
}

bool f32_takes_windowed(int d, int B, int H, int H0, int N) {
  return d == 64 && H0 > 0 && H0 < H && N > 0 && B > 0 && f32_window_rows((int64_t)B * H0, N) == 64 &&
         (int64_t)B * H0 * ((N + 63) / 64) < (1 << 22) && (int64_t)B * (H - H0) < (1 << 20);
}

hipError_t launch_linear_f32(const AttnArgs& a, bool with_windowed, hipStream_t s) {
  if (a.H - a.H0 <= 0 || a.N <= 0 || a.B <= 0) return hipSuccess;
  return a.d == 64 ? forward<64>(a, with_windowed, s) : forward<128>(a, false, s);
}
hipError_t launch_linear_backward_f32(const BwdArgs& a, bool with_windowed, hipStream_t s) {
  if (a.H - a.H0 <= 0 || a.N <= 0 || a.B <= 0) return hipSuccess;
  return a.d == 64 ? backward<64>(a, with_windowed, s) : backward<128>(a, false, s);
}

}  // namespace gformer
