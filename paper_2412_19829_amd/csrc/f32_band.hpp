// One workgroup's work for the windowed heads in single precision (f32_windowed.hip describes it), as device
// functions: the kernels of its own run them, and so do the blocks behind the linear heads' in the launches
// that hold both (f32_linear.hip).
#pragma once

#include "common.hpp"
#include "f32_mfma.hpp"
#include "mfma.hpp"

namespace gformer {
namespace {

constexpr int kF32Tile = 64;      // band rows per LDS tile
constexpr int kF32BandThreads = 256;
constexpr int kF32Xcds = 8;

// Staging of one tensor's tile: thread t moves 16-byte pieces (row t / (D/4) + i * RP).
template <int D> struct F32Stage {
  static constexpr int C4 = D / 4, RP = kF32BandThreads / C4, PIECES = kF32Tile / RP;
  int row, col;
  __device__ __forceinline__ explicit F32Stage(int tid) : row(tid / C4), col(4 * (tid % C4)) {}
  // rows past N - 1 re-read row N - 1 (in bounds; never visible).  (A uniform base and 32-bit offsets under a clamp, which
  // the linear walks gain by, cost this one: training steps of windowed heads 7 x 8 x 1242 x 64 155.3 -> 157.0 us, 4 x
  // (2 + 10) x 876 150.8 -> 153.0, 4 x (3 + 13) x 2048 269.7 -> 271.8.)
  __device__ __forceinline__ void load(f32x4 (&dst)[PIECES], const float* base, int64_t sn, int t0, int N) const {
#pragma unroll
    for (int i = 0; i < PIECES; ++i)
      dst[i] = *reinterpret_cast<const f32x4*>(base + (int64_t)min(t0 + row + i * RP, N - 1) * sn + col);
  }
  __device__ __forceinline__ void store(float* tile, const f32x4 (&src)[PIECES]) const {
#pragma unroll
    for (int i = 0; i < PIECES; ++i)
      *reinterpret_cast<f32x4*>(tile + (row + i * RP) * kF32Row<D> + col) = src[i];
  }
  // true when one of the thread's values is an infinity or a NaN
  static __device__ __forceinline__ bool not_finite(const f32x4 (&src)[PIECES]) {
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < PIECES; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) t = fmaf(src[i][j], 0.f, t);
    return t != 0.f;
  }
};

template <int D> struct F32WinSmem {
  float x[kF32Tile * kF32Row<D>];   // K (queries resident) or Q (keys resident)
  float y[kF32Tile * kF32Row<D>];   // V or dO
  float stat[kF32Tile * 2];         // (lse, D) of the tile's queries
  float red[4][4][16];           // per-wave statistics on their way to the other waves
  int bad[2];                    // tile holds an infinity or a NaN (alternating between tiles)
};

// acc[4*hh + x] += (rows of one group of 16 band rows)^T w: w[r] is the weight of band row 4*g + r for
// this lane's resident row, seen[r] whether that row is visible at all.
template <int D>
__device__ __forceinline__ void add_weighted(f32x4 (&acc)[D / 16], const float* rows, const float (&w)[4],
                                             const bool (&seen)[4], int lane, bool bad) {
  const int g = lane >> 4, i = lane & 15;
  if (!bad) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int hh = 0; hh < D / 64; ++hh) {
        const f32x4 x = lds4(rows + (4 * g + r) * kF32Row<D> + 64 * hh + 4 * i);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[4 * hh + j] = mfma_f32(x[j], w[r], acc[4 * hh + j]);
      }
    return;
  }
  for (int k = 0; k < 16; ++k) {
    float wk = 0.f;
    bool sk = false;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float wr = __shfl(w[r], 16 * (k / 4) + i, 64);
      const bool sr = __shfl((int)seen[r], 16 * (k / 4) + i, 64) != 0;
      if (k % 4 == r) { wk = wr; sk = sr; }
    }
    if (sk) {
#pragma unroll
      for (int hh = 0; hh < D / 64; ++hh)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const f32x4 x = lds4(rows + k * kF32Row<D> + 64 * hh + 16 * g + 4 * r);
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[4 * hh + j][r] = fmaf(wk, x[j], acc[4 * hh + j][r]);
        }
    }
  }
}

// Row `idx` of the block: element 4*kk + j of the lane is column 16*kk + 4*g + j.
template <int D>
__device__ __forceinline__ void load_resident(float (&dst)[D / 4], const float* row, int lane) {
  const int g = lane >> 4;
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(row + 16 * kk + 4 * g);
#pragma unroll
    for (int j = 0; j < 4; ++j) dst[4 * kk + j] = x[j];
  }
}

// (row block, head, batch) of a workgroup: neighbouring blocks of a head share most of their band,
// so each XCD (own L2) gets one contiguous run of the logical order.
__device__ __forceinline__ void block_of(int nblk, int heads, int batch, int block, int& blk, int& h, int& b) {
  const int total = nblk * heads * batch, per = total / kF32Xcds, rem = total % kF32Xcds;
  const int xcd = block % kF32Xcds, slot = block / kF32Xcds;
  const int lb = xcd * per + min(xcd, rem) + slot;
  blk = lb % nblk;
  h = (lb / nblk) % heads;
  b = lb / (nblk * heads);
}

// acc of the 4 / QB waves that share their resident rows -> their sum, times `f`, written as rows.
// Lane l holds columns 64*hh + 16*g + 4*r + x of row l%16 in acc[4*hh + x][r].
template <int D, int QB>
__device__ __forceinline__ void write_rows(const f32x4 (&acc)[D / 16], float f, float* tiles, float* out,
                                           int64_t sn, int row0, int N, int tid) {
  const int lane = tid & 63, wave = tid >> 6, g = lane >> 4, i = lane & 15;
  if constexpr (QB == 4) {
    if (row0 + i < N) {
      float* o = out + (int64_t)(row0 + i) * sn + 16 * g;
#pragma unroll
      for (int hh = 0; hh < D / 64; ++hh)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          *reinterpret_cast<f32x4*>(o + 64 * hh + 4 * r) =
              f32x4{acc[4 * hh][r] * f, acc[4 * hh + 1][r] * f, acc[4 * hh + 2][r] * f, acc[4 * hh + 3][r] * f};
    }
  } else {
    static_assert(QB == 1, "four waves hold their own rows or share one group of 16");
    lds_barrier();   // every wave is done with the tiles
    float* mine = tiles + (wave * 16 + i) * kF32Row<D> + 16 * g;
#pragma unroll
    for (int hh = 0; hh < D / 64; ++hh)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        *reinterpret_cast<f32x4*>(mine + 64 * hh + 4 * r) =
            f32x4{acc[4 * hh][r] * f, acc[4 * hh + 1][r] * f, acc[4 * hh + 2][r] * f, acc[4 * hh + 3][r] * f};
    lds_barrier();
    for (int p = tid; p < 16 * D / 4; p += kF32BandThreads) {
      const int row = p / (D / 4), col = 4 * (p % (D / 4));
      if (row0 + row < N) {
        f32x4 s = lds4(tiles + row * kF32Row<D> + col);
#pragma unroll
        for (int w = 1; w < 4; ++w) s += lds4(tiles + (w * 16 + row) * kF32Row<D> + col);
        *reinterpret_cast<f32x4*>(out + (int64_t)(row0 + row) * sn + col) = s;
      }
    }
  }
}

// Walks the band [lo, hi] in tiles of 64 rows of x and y: body(t0, bad) between barriers, the next
// tile's loads in flight meanwhile.
template <int D, bool CHECK_X, bool CHECK_Y, typename Extra, typename Body>
__device__ __forceinline__ void walk_band(F32WinSmem<D>& sm, const float* xb, int64_t xsn, const float* yb,
                                          int64_t ysn, int lo, int hi, int N, int tid, Extra extra, Body body) {
  // d = 128: a tile on its way in registers beside the resident rows and the accumulators would
  // spill; the other workgroup of the compute unit covers the wait instead
  constexpr bool AHEAD = D == 64;
  const F32Stage<D> st(tid);
  f32x4 xr[F32Stage<D>::PIECES], yr[F32Stage<D>::PIECES];
  if (tid < 2) sm.bad[tid] = 0;
  if (AHEAD) {
    st.load(xr, xb, xsn, lo, N);
    st.load(yr, yb, ysn, lo, N);
  }
  int it = 0;
  for (int t0 = lo; t0 <= hi; t0 += kF32Tile, ++it) {
    if (!AHEAD) {
      st.load(xr, xb, xsn, t0, N);
      st.load(yr, yb, ysn, t0, N);
    }
    lds_barrier();   // the tile before is consumed (first round: the flags are clear)
    st.store(sm.x, xr);
    st.store(sm.y, yr);
    if ((CHECK_X && F32Stage<D>::not_finite(xr)) || (CHECK_Y && F32Stage<D>::not_finite(yr)))
      sm.bad[it & 1] = 1;
    extra(t0);
    if (AHEAD && t0 + kF32Tile <= hi) {
      st.load(xr, xb, xsn, t0 + kF32Tile, N);
      st.load(yr, yb, ysn, t0 + kF32Tile, N);
    }
    lds_barrier();
    const bool bad = __builtin_amdgcn_readfirstlane(sm.bad[it & 1]) != 0;   // uniform
    if (tid == 0) sm.bad[(it + 1) & 1] = 0;   // read last in the round before this one
    body(t0, bad);
  }
}

// ---- forward ---------------------------------------------------------------------------------
template <int D, int QB>
__device__ __forceinline__ void windowed_f32(const AttnArgs& a, int block, unsigned char* smem_raw) {
  constexpr int KS = 4 / QB;
  F32WinSmem<D>& sm = *reinterpret_cast<F32WinSmem<D>*>(smem_raw);
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, i = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = a.N;
  int blk, h, b;
  block_of((N + 16 * QB - 1) / (16 * QB), a.H0, a.B, block, blk, h, b);
  const float* qp = reinterpret_cast<const float*>(a.q.base) + b * a.q.sb + h * a.q.sh;
  const float* kp = reinterpret_cast<const float*>(a.k.base) + b * a.k.sb + h * a.k.sh;
  const float* vp = reinterpret_cast<const float*>(a.v.base) + b * a.v.sb + h * a.v.sh;
  float* op = reinterpret_cast<float*>(a.out) + b * a.osb + h * a.osh;
  const int i0 = blk * 16 * QB;
  const int q0 = i0 + 16 * (wave % QB), ks = wave / QB;
  const int wl = a.wleft, wr = a.wright;
  float qreg[D / 4];
  load_resident<D>(qreg, qp + (int64_t)min(q0 + i, N - 1) * a.q.sn, lane);
  f32x4 acc[D / 16];
#pragma unroll
  for (int t = 0; t < D / 16; ++t) acc[t] = kZeroF4;
  float m = -INFINITY, l = 0.f;   // l: this lane's keys only
  const int lo = max(0, i0 - wl) & ~15, hi = min(N - 1, i0 + 16 * QB - 1 + wr);
  const int qi = q0 + i;
  const int klo = qi - wl, khi = min(qi + wr, N - 1);   // this lane's query sees keys klo..khi
  walk_band<D, false, true>(sm, kp, a.k.sn, vp, a.v.sn, lo, hi, N, tid, [](int) {}, [&](int t0, bool bad) {
    float p[4][4];
    bool seen[4][4];
    bool act[4];
    float mx = -INFINITY;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k0 = t0 + 16 * s;
      act[s] = s % KS == ks && k0 <= min(q0 + 15 + wr, N - 1) && k0 + 15 >= q0 - wl;   // wave-uniform
      if (act[s]) {
        const f32x4 sc = rows_product<D>(sm.x + (16 * s + i) * kF32Row<D> + 4 * g, qreg);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int key = k0 + 4 * g + r;
          seen[s][r] = key >= klo && key <= khi;
          p[s][r] = seen[s][r] ? sc[r] * a.scale : -INFINITY;
          mx = fmaxf(mx, p[s][r]);
        }
      }
    }
    if (!(act[0] || act[1] || act[2] || act[3])) return;
    const float m_new = fmaxf(m, max_over_groups(mx));
    const float m_use = m_new == -INFINITY ? 0.f : m_new;   // no visible key so far
    const float alpha = expf(m - m_use);                     // exp(-inf) = 0 before the first one
    m = m_new;
    l *= alpha;
#pragma unroll
    for (int t = 0; t < D / 16; ++t) acc[t] *= alpha;
#pragma unroll
    for (int s = 0; s < 4; ++s)
      if (act[s]) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          p[s][r] = seen[s][r] ? expf(p[s][r] - m_use) : 0.f;
          l += p[s][r];
        }
        add_weighted<D>(acc, sm.y + 16 * s * kF32Row<D>, p[s], seen[s], lane, bad);
      }
  });
  l = sum_over_groups(l);
  float f;
  if constexpr (KS == 1) {
    f = 1.f / l;
  } else {
    // the waves' sums meet under their largest maximum
    if (g == 0) { sm.red[wave][0][i] = m; sm.red[wave][1][i] = l; }
    lds_barrier();
    float mt = -INFINITY, lt = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) mt = fmaxf(mt, sm.red[w][0][i]);
    const float m_use = mt == -INFINITY ? 0.f : mt;
#pragma unroll
    for (int w = 0; w < 4; ++w) lt += sm.red[w][1][i] * expf(sm.red[w][0][i] - m_use);
    f = expf(m - m_use) / lt;
  }
  write_rows<D, QB>(acc, f, sm.x, op, a.osn, q0, N, tid);
}

// ---- backward: per query, (lse_i, D_i) into the workspace and dq_i ----------------------------
// Two walks over the band: the row's maximum, sum and D_i = sum_j p_ij dO_i.v_j, then ds and its
// product with the keys (five products of the nine of the whole backward pass).
template <int D, int QB>
__device__ __forceinline__ void windowed_bwd_q_f32(const BwdArgs& a, int block, unsigned char* smem_raw) {
  constexpr int KS = 4 / QB;
  F32WinSmem<D>& sm = *reinterpret_cast<F32WinSmem<D>*>(smem_raw);
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, i = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = a.N;
  int blk, h, b;
  block_of((N + 16 * QB - 1) / (16 * QB), a.H0, a.B, block, blk, h, b);
  const float* qp = reinterpret_cast<const float*>(a.q.base) + b * a.q.sb + h * a.q.sh;
  const float* kp = reinterpret_cast<const float*>(a.k.base) + b * a.k.sb + h * a.k.sh;
  const float* vp = reinterpret_cast<const float*>(a.v.base) + b * a.v.sb + h * a.v.sh;
  const float* dp = reinterpret_cast<const float*>(a.dout.base) + b * a.dout.sb + h * a.dout.sh;
  float* ws = a.ws + ((int64_t)b * a.H + h) * N * 2;
  const int i0 = blk * 16 * QB;
  const int q0 = i0 + 16 * (wave % QB), ks = wave / QB;
  const int wl = a.wleft, wr = a.wright;
  float qreg[D / 4], dreg[D / 4];
  {
    const int64_t row = min(q0 + i, N - 1);
    load_resident<D>(qreg, qp + row * a.q.sn, lane);
    load_resident<D>(dreg, dp + row * a.dout.sn, lane);
  }
  const int lo = max(0, i0 - wl) & ~15, hi = min(N - 1, i0 + 16 * QB - 1 + wr);
  const int qi = q0 + i;
  const int klo = qi - wl, khi = min(qi + wr, N - 1);
  auto active = [&](int s, int t0) {
    const int k0 = t0 + 16 * s;
    return s % KS == ks && k0 <= min(q0 + 15 + wr, N - 1) && k0 + 15 >= q0 - wl;   // wave-uniform
  };
  float m = -INFINITY, l = 0.f, dsum = 0.f;
  walk_band<D, false, false>(sm, kp, a.k.sn, vp, a.v.sn, lo, hi, N, tid, [](int) {}, [&](int t0, bool) {
    float sc[4][4], dv[4][4];
    float mx = -INFINITY;
    bool any = false;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
#pragma unroll
      for (int r = 0; r < 4; ++r) { sc[s][r] = -INFINITY; dv[s][r] = 0.f; }
      if (active(s, t0)) {
        any = true;
        const int off = (16 * s + i) * kF32Row<D> + 4 * g;
        const f32x4 x = rows_product<D>(sm.x + off, qreg), y = rows_product<D>(sm.y + off, dreg);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int key = t0 + 16 * s + 4 * g + r;
          const bool seen = key >= klo && key <= khi;
          sc[s][r] = seen ? x[r] * a.scale : -INFINITY;
          dv[s][r] = seen ? y[r] : 0.f;
          mx = fmaxf(mx, sc[s][r]);
        }
      }
    }
    if (!any) return;
    const float m_new = fmaxf(m, max_over_groups(mx));
    const float m_use = m_new == -INFINITY ? 0.f : m_new;
    const float alpha = expf(m - m_use);
    m = m_new;
    l *= alpha;
    dsum *= alpha;
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float p = expf(sc[s][r] - m_use);   // 0 where nothing is seen
        l += p;
        dsum = fmaf(p, dv[s][r], dsum);
      }
  });
  l = sum_over_groups(l);
  dsum = sum_over_groups(dsum);
  if constexpr (KS > 1) {
    if (g == 0) { sm.red[wave][0][i] = m; sm.red[wave][1][i] = l; sm.red[wave][2][i] = dsum; }
    lds_barrier();
    float mt = -INFINITY;
#pragma unroll
    for (int w = 0; w < 4; ++w) mt = fmaxf(mt, sm.red[w][0][i]);
    const float m_use = mt == -INFINITY ? 0.f : mt;
    float lt = 0.f, dt = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float e = expf(sm.red[w][0][i] - m_use);
      lt = fmaf(sm.red[w][1][i], e, lt);
      dt = fmaf(sm.red[w][2][i], e, dt);
    }
    m = mt; l = lt; dsum = dt;
  }
  const float inv = 1.f / l, Di = dsum * inv;
  if (ks == 0 && g == 0 && qi < N) {
    ws[2 * (int64_t)qi] = m + logf(l);
    ws[2 * (int64_t)qi + 1] = Di;
  }
  f32x4 acc[D / 16];
#pragma unroll
  for (int t = 0; t < D / 16; ++t) acc[t] = kZeroF4;
  lds_barrier();   // the last tile of the first walk is consumed, its flags may be cleared
  walk_band<D, true, false>(sm, kp, a.k.sn, vp, a.v.sn, lo, hi, N, tid, [](int) {}, [&](int t0, bool bad) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
      if (active(s, t0)) {
        const int off = (16 * s + i) * kF32Row<D> + 4 * g;
        const f32x4 x = rows_product<D>(sm.x + off, qreg), y = rows_product<D>(sm.y + off, dreg);
        float ds[4];
        bool seen[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int key = t0 + 16 * s + 4 * g + r;
          seen[r] = key >= klo && key <= khi;
          ds[r] = seen[r] ? expf(x[r] * a.scale - m) * inv * (y[r] - Di) : 0.f;
        }
        add_weighted<D>(acc, sm.x + 16 * s * kF32Row<D>, ds, seen, lane, bad);
      }
  });
  write_rows<D, QB>(acc, a.scale, sm.x, reinterpret_cast<float*>(a.dq) + b * a.q.sb + h * a.q.sh, a.q.sn, q0, N, tid);
}

// ---- backward: per key, dk_j and dv_j over the queries that see it -----------------------------
template <int D, int QB>
__device__ __forceinline__ void windowed_bwd_kv_f32(const BwdArgs& a, int block, unsigned char* smem_raw) {
  constexpr int KS = 4 / QB;
  F32WinSmem<D>& sm = *reinterpret_cast<F32WinSmem<D>*>(smem_raw);
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, i = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = a.N;
  int blk, h, b;
  block_of((N + 16 * QB - 1) / (16 * QB), a.H0, a.B, block, blk, h, b);
  const float* qp = reinterpret_cast<const float*>(a.q.base) + b * a.q.sb + h * a.q.sh;
  const float* kp = reinterpret_cast<const float*>(a.k.base) + b * a.k.sb + h * a.k.sh;
  const float* vp = reinterpret_cast<const float*>(a.v.base) + b * a.v.sb + h * a.v.sh;
  const float* dp = reinterpret_cast<const float*>(a.dout.base) + b * a.dout.sb + h * a.dout.sh;
  const float* ws = a.ws + ((int64_t)b * a.H + h) * N * 2;
  const int j0 = blk * 16 * QB;
  const int k0 = j0 + 16 * (wave % QB), ks = wave / QB;
  const int wl = a.wleft, wr = a.wright;
  float kreg[D / 4], vreg[D / 4];
  {
    const int64_t row = min(k0 + i, N - 1);
    load_resident<D>(kreg, kp + row * a.k.sn, lane);
    load_resident<D>(vreg, vp + row * a.v.sn, lane);
  }
  f32x4 acck[D / 16], accv[D / 16];
#pragma unroll
  for (int t = 0; t < D / 16; ++t) { acck[t] = kZeroF4; accv[t] = kZeroF4; }
  const int kj = k0 + i;
  const int qlo = kj - wr, qhi = min(kj + wl, N - 1);   // key kj is seen by queries qlo..qhi
  const int lo = max(0, j0 - wr) & ~15, hi = min(N - 1, j0 + 16 * QB - 1 + wl);
  auto stats = [&](int t0) {
    if (tid < kF32Tile) {
      const float2 s = *reinterpret_cast<const float2*>(ws + 2 * (int64_t)min(t0 + tid, N - 1));
      sm.stat[tid] = s.x;
      sm.stat[kF32Tile + tid] = s.y;
    }
  };
  walk_band<D, true, true>(sm, qp, a.q.sn, dp, a.dout.sn, lo, hi, N, tid, stats, [&](int t0, bool bad) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int r0 = t0 + 16 * s;
      if (s % KS == ks && r0 <= min(k0 + 15 + wl, N - 1) && r0 + 15 >= k0 - wr) {   // wave-uniform
        const int off = (16 * s + i) * kF32Row<D> + 4 * g;
        const f32x4 x = rows_product<D>(sm.x + off, kreg), y = rows_product<D>(sm.y + off, vreg);
        const f32x4 lse = lds4(sm.stat + 16 * s + 4 * g), Di = lds4(sm.stat + kF32Tile + 16 * s + 4 * g);
        float p[4], ds[4];
        bool seen[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int q = r0 + 4 * g + r;
          seen[r] = q >= qlo && q <= qhi;
          p[r] = seen[r] ? expf(x[r] * a.scale - lse[r]) : 0.f;
          ds[r] = seen[r] ? p[r] * (y[r] - Di[r]) : 0.f;
        }
        add_weighted<D>(accv, sm.y + 16 * s * kF32Row<D>, p, seen, lane, bad);
        add_weighted<D>(acck, sm.x + 16 * s * kF32Row<D>, ds, seen, lane, bad);
      }
    }
  });
  write_rows<D, QB>(acck, a.scale, sm.x, reinterpret_cast<float*>(a.dk) + b * a.k.sb + h * a.k.sh, a.k.sn, k0, N, tid);
  write_rows<D, QB>(accv, 1.f, sm.x, reinterpret_cast<float*>(a.dv) + b * a.v.sb + h * a.v.sh, a.v.sn, k0, N, tid);
}

}  // namespace
}  // namespace gformer
