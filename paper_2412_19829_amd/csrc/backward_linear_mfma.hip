// Backward pass of the causal linear-attention heads on bf16 matrix cores (section II-B's ratio
// and Algorithm 1's running sums, differentiated; the formulas are stated at the top of
// backward_scalar.hip).
//
// With fq = phi(q), fk = phi(k), A_i = sum_{j<=i} fk_j v_j^T, Z_i = sum_{j<=i} fk_j,
// den_i = fq_i.Z_i + eps, g_i = dO_i / den_i, c_i = g_i.(fq_i^T A_i) / den_i:
//   dfq_i = A_i g_i - c_i Z_i,
//   dfk_j = B_j v_j - Y_j,  dv_j = B_j^T fk_j,   B_j = sum_{i>=j} fq_i g_i^T,  Y_j = sum_{i>=j} c_i fq_i.
// In chunks of 64 tokens, with S = tril(fq fk^T), T = tril(dO v^T), T' = T / den - tril(c 1^T) (row i, column j <= i)
// and the sums (A, Z) over earlier chunks, (B, Y) over later chunks:
//   forward scan:  r = A dO,  den = rowsum(S) + fq.Z + eps,  c = (fq.r + rowsum(S * T)) / den^2 (which is
//                  dO.num / den^2 without a numerator),  dfq = T' fk + r / den - c Z^T;   then A += fk^T v, Z += colsum(fk)
//   reverse scan:  dfk = T'^T fq + v B^T - 1 Y^T,  dv = (S / den)^T dO + fk B;   then B += fq^T dO / den, Y += fq^T c
// What bounds them: the phases of the one workgroup a unit, one after the other, of whose cycles
// the LDS pipeline takes 45 and 50 %, a fifth of that in conflicts, the vector unit 40 %, the matrix core 15 %; and 13.3 tensors' worth of traffic (the scans' eight reads and three writes, and what light rounds
// read again) at 4.0 (forward) and 4.1 TB/s (reverse) on 128 heads x 8192, of the 4.9 a copy reaches.  With the
// numerator as two products of its own (S as a pair), dO and dO / den as tiles of their own, the 32 x 32 tile above the
// diagonal computed and multiplied, and the column sums read from LDS element by element, the same scans took 953 us
// (841 without, 826 with the feature map as a maximum; 4 x (6 + 26) heads x 8192 with the windowed heads 1083 and 1000; 32 x 1000
// 81.5 and 72.0).  Row stores behind the next chunk's staging and loads instead of in front of it: 883.  Of a forward chunk 25 %
// go to (a), where three waves work twice as long as the others, 22 to (b) and (c), 16 to (d), 37 to (e).
// These are the kernels of d = 128, and of d = 64 where the workspace holds no segment sums.
// One workgroup per (batch, head), segment and scan: with fewer heads than compute units a head
// is cut into up to four segments, and a workgroup first sums the chunks in front of (behind)
// its segment in light rounds (the update of the carried sums alone) before it scans the segment.
// Every product is a 32x32 MFMA tile job handed out
// over the waves; the chunk's tiles sit in LDS row-major with a row stride that serves both the
// row read (contraction over the feature/value index) and the transpose read (contraction over
// tokens); the carried d x d sum lives in fp32 accumulators spread over the waves, with a bf16
// copy in LDS as the operand of the next chunk's products; Z, Y, den and c stay in fp32.
// The forward scan leaves (den_i, c_i) in the workspace for the reverse scan.
#include "backward_band.hpp"
#include "backward_linear_common.hpp"

namespace gformer {
namespace {

// T' is a difference of two nearly equal terms and a gradient row sums it against phi with
// signs: its rounding to one bf16 is the largest single error of these kernels.  It is therefore
// kept as a pair, bf16(T') in `tp` and bf16(T' - bf16(T')) in `tl` (16 mantissa bits), and every
// product with T' runs over both.  S and T enter den and c, which enter every T' of their row, as the fp32
// products they are; dv = S^T g in the reverse scan takes S as one bf16 (its rows do not cancel).
template <int D> struct LbSmemBase {
  using C = LbCfg<D>;
  uint16_t fq[CH * C::R], fk[CH * C::R], v[CH * C::R], g[CH * C::R];
  uint16_t st[D * C::R];              // bf16 copy of the carried sum, [feature][value]
  uint16_t tp[CH * SR], tl[CH * SR];  // T' (forward scan: [i][j]; reverse scan: [j][i]), its low half
  float z[D];                         // Z (forward scan) or Y (reverse scan)
  float zpart[C::MT][D];
};
template <int D> struct LbSmem : LbSmemBase<D> {
  float part[2][3][32];               // row sums of S and of S * T per 32 x 32 tile on or below the diagonal
  float red[2][LbCfg<D>::MT][CH];     // phi(q).(A dO) and phi(q).Z per feature block
};

// the reverse scan scales by 1/den where a product needs it and keeps dO itself in the tile `g`: T' is formed as
// (dO.v)/den - c in fp32, exactly as the forward scan forms c, so that the two cancel where they must (a token that
// only sees itself).
template <int D> struct LbSmemKv : LbSmemBase<D> {
  uint16_t sm[CH * SR];               // S / den, [j][i]
  float dz[CH], den[CH], cc[CH];      // den: the reciprocal
};
static_assert(sizeof(LbSmemKv<128>) <= 160 * 1024 && sizeof(LbSmem<128>) <= 160 * 1024,
              "one workgroup's tiles must fit the LDS of a compute unit");

// Sum over this lane's eight tokens of w * operand, w in fp32.
__device__ __forceinline__ float weighted8(bf16x8 x, const float* w, float acc) {
  const u32x4 u = as_u32x4(x);
  const float4 a = *reinterpret_cast<const float4*>(w), b = *reinterpret_cast<const float4*>(w + 4);
  acc = fmaf(bf16_lo(u[0]), a.x, fmaf(bf16_hi(u[0]), a.y, acc));
  acc = fmaf(bf16_lo(u[1]), a.z, fmaf(bf16_hi(u[1]), a.w, acc));
  acc = fmaf(bf16_lo(u[2]), b.x, fmaf(bf16_hi(u[2]), b.y, acc));
  return fmaf(bf16_lo(u[3]), b.z, fmaf(bf16_hi(u[3]), b.w, acc));
}
__device__ __forceinline__ float sum8(bf16x8 x, float acc) {
  const u32x4 u = as_u32x4(x);
#pragma unroll
  for (int w = 0; w < 4; ++w) acc = dot2_ones_bf16(u[w], acc);
  return acc;
}
// The operand with each of its eight tokens scaled.
__device__ __forceinline__ bf16x8 scaled8(bf16x8 x, const float* w) {
  const u32x4 u = as_u32x4(x);
  const float4 a = *reinterpret_cast<const float4*>(w), b = *reinterpret_cast<const float4*>(w + 4);
  u32x4 o;
  o[0] = pack_bf16(bf16_lo(u[0]) * a.x, bf16_hi(u[0]) * a.y);
  o[1] = pack_bf16(bf16_lo(u[1]) * a.z, bf16_hi(u[1]) * a.w);
  o[2] = pack_bf16(bf16_lo(u[2]) * b.x, bf16_hi(u[2]) * b.y);
  o[3] = pack_bf16(bf16_lo(u[3]) * b.z, bf16_hi(u[3]) * b.w);
  return as_bf16x8(o);
}
// Carried sum, tile u of a wave: value block vt, feature block ft0 + u.  The waves of a feature block share the column
// sums of a chunk: each adds up the operand of the steps kk with kk % MT == vt, picked out with wave-uniform selects
// (a branch there splits the products' schedule: 1003 against 1001 us, 725 against 700 on short heads).
template <int D> struct SumTiles {
  int vt, ft0;
  __device__ __forceinline__ explicit SumTiles(int wave) : vt(wave * LbCfg<D>::TPW / LbCfg<D>::MT), ft0(wave * LbCfg<D>::TPW % LbCfg<D>::MT) {}
  static constexpr int STEPS = CH / 16 / LbCfg<D>::MT;   // steps a wave adds up: kk = x * MT + vt
  struct Picked { bf16x8 x[STEPS]; };
  __device__ __forceinline__ void pick(Picked& p, int kk, bf16x8 op) const {
    constexpr int MT = LbCfg<D>::MT;
    p.x[kk / MT] = kk % MT == 0 || kk % MT == vt ? op : p.x[kk / MT];
  }
  __device__ __forceinline__ float sum(const Picked& p, float acc) const {
#pragma unroll
    for (int x = 0; x < STEPS; ++x) acc = sum8(p.x[x], acc);
    return acc;
  }
  __device__ __forceinline__ float sum(const Picked& p, const float* weights, int lh, float acc) const {
#pragma unroll
    for (int x = 0; x < STEPS; ++x) acc = weighted8(p.x[x], weights + 16 * (x * LbCfg<D>::MT + vt) + 8 * lh, acc);
    return acc;
  }
  // the lane's column sums of its feature blocks for the other waves
  __device__ __forceinline__ void put(float (&zpart)[LbCfg<D>::MT][D], const float (&zs)[LbCfg<D>::TPW], int ln, int lh) const {
#pragma unroll
    for (int u = 0; u < LbCfg<D>::TPW; ++u) {
      const float z = sum_over_halves(zs[u]);
      if (lh == 0) zpart[vt][32 * (ft0 + u) + ln] = z;
    }
  }
  // bf16 copy of the sums, the operand of the next chunk's products
  __device__ __forceinline__ void copy(uint16_t* st, const f32x16 (&sacc)[LbCfg<D>::TPW], int ln, int lh) const {
#pragma unroll
    for (int u = 0; u < LbCfg<D>::TPW; ++u)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4)
        put4(&st[(32 * (ft0 + u) + ln) * LbCfg<D>::R + 32 * vt + 8 * g4 + 4 * lh], sacc[u][4 * g4 + 0],
             sacc[u][4 * g4 + 1], sacc[u][4 * g4 + 2], sacc[u][4 * g4 + 3]);
  }
};

// ---------------------------------------------------------------------------------------
// forward scan: dq, and (den_i, c_i) into the workspace
// ---------------------------------------------------------------------------------------
template <int D, bool ELU1>
__device__ __forceinline__ void scan_q(const BwdArgs& a, int h, int b, int seg, unsigned char* smem_raw) {
  using C = LbCfg<D>;
  constexpr int MT = C::MT, KS = C::KS, NT = C::NT, R = C::R, TPW = C::TPW, PCS = C::PCS;
  LbSmem<D>& sm = *reinterpret_cast<LbSmem<D>*>(smem_raw);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, ln = lane & 31, lh = lane >> 5;
  const HeadCtx<D> hc = head_ctx<D>(a, b, h);
  uint16_t* dqp = reinterpret_cast<uint16_t*>(a.dq) + b * a.q.sb + h * a.q.sh;
  const int N = a.N;
  // this workgroup writes the chunks [cb, ce) of its head; the chunks in front of them are only
  // summed (light rounds: the state update alone)
  const int cb = a.lin_bounds[seg], ce = a.lin_bounds[seg + 1];
  if (cb >= ce) return;
  const int trl = lds_operand_tr_lane_offset(R, lane) + 8 * lh * R;

  u32x4 rq[PCS], rk[PCS], rv[PCS], rdo[PCS];
  auto load_chunk = [&](int n) {
    const bool full = n >= cb;   // uniform
#pragma unroll
    for (int i = 0; i < PCS; ++i) {
      const int p = tid + i * NT, row = p / C::C8, col = 8 * (p % C::C8);
      const int64_t tok = min(n * CH + row, N - 1);
      rk[i] = *reinterpret_cast<const u32x4*>(hc.k + tok * a.k.sn + col);
      rv[i] = *reinterpret_cast<const u32x4*>(hc.v + tok * a.v.sn + col);
      if (full) {
        rq[i] = *reinterpret_cast<const u32x4*>(hc.q + tok * a.q.sn + col);
        rdo[i] = *reinterpret_cast<const u32x4*>(hc.dout + tok * a.dout.sn + col);
      }
    }
  };
  // the feature map, in place in the staging registers (light rounds: only the tensor they read)
  auto map_chunk = [&](int n) {
    const bool full = n >= cb;
#pragma unroll
    for (int i = 0; i < PCS; ++i) {
      rk[i] = map8<ELU1>(rk[i]);
      if (full) rq[i] = map8<ELU1>(rq[i]);
    }
  };
  auto stage_chunk = [&](int n) {
    const bool full = n >= cb;
#pragma unroll
    for (int i = 0; i < PCS; ++i) {
      const int p = tid + i * NT, row = p / C::C8, col = 8 * (p % C::C8);
      const bool valid = n * CH + row < N;   // rows past the end become zeros: they contribute nothing
      *reinterpret_cast<u32x4*>(&sm.fk[row * R + col]) = valid ? rk[i] : kZero4;
      *reinterpret_cast<u32x4*>(&sm.v[row * R + col]) = valid ? rv[i] : kZero4;
      if (full) {
        *reinterpret_cast<u32x4*>(&sm.fq[row * R + col]) = valid ? rq[i] : kZero4;
        *reinterpret_cast<u32x4*>(&sm.g[row * R + col]) = valid ? rdo[i] : kZero4;   // dO
      }
    }
  };

  const SumTiles<D> tiles(wave);   // carried sum A^T in accumulators
  f32x16 sacc[TPW];
#pragma unroll
  for (int u = 0; u < TPW; ++u)
#pragma unroll
    for (int r = 0; r < 16; ++r) sacc[u][r] = 0.f;
  for (int i = tid; i < D * R / 2; i += NT) reinterpret_cast<uint32_t*>(sm.st)[i] = 0u;
  if (tid < D) sm.z[tid] = 0.f;

  // Light rounds, two chunks at a time: the chunks in front of the segment only feed the carried
  // sums, so phi(K) and V of chunk n go to the fk / v tiles and those of chunk n + 1 to the fq / g
  // tiles (and travel in the q / dO staging registers), one barrier pair for both.
  auto load_pair = [&](int n) {
#pragma unroll
    for (int i = 0; i < PCS; ++i) {
      const int p = tid + i * NT, row = p / C::C8, col = 8 * (p % C::C8);
      const int64_t t0 = min(n * CH + row, N - 1), t1 = min((n + 1) * CH + row, N - 1);
      rk[i] = *reinterpret_cast<const u32x4*>(hc.k + t0 * a.k.sn + col);
      rv[i] = *reinterpret_cast<const u32x4*>(hc.v + t0 * a.v.sn + col);
      rq[i] = *reinterpret_cast<const u32x4*>(hc.k + t1 * a.k.sn + col);
      rdo[i] = *reinterpret_cast<const u32x4*>(hc.v + t1 * a.v.sn + col);
    }
  };
  int n0 = 0;   // first chunk of the round-by-round loop below
  if (cb >= 2) {
    load_pair(0);
    for (; n0 + 2 <= cb; n0 += 2) {
      // chunks in front of a segment are whole: no rows past the end here
#pragma unroll
      for (int i = 0; i < PCS; ++i) {
        const int p = tid + i * NT, row = p / C::C8, col = 8 * (p % C::C8);
        *reinterpret_cast<u32x4*>(&sm.fk[row * R + col]) = map8<ELU1>(rk[i]);
        *reinterpret_cast<u32x4*>(&sm.v[row * R + col]) = rv[i];
        *reinterpret_cast<u32x4*>(&sm.fq[row * R + col]) = map8<ELU1>(rq[i]);
        *reinterpret_cast<u32x4*>(&sm.g[row * R + col]) = rdo[i];
      }
      if (n0 + 4 <= cb) load_pair(n0 + 2);
      lds_barrier();
      float zs[TPW];
      typename SumTiles<D>::Picked z0[TPW], z1[TPW];
#pragma unroll
      for (int kk = 0; kk < CH / 16; ++kk) {
        const bf16x8 v0 = col_op(sm.v + trl, R, 16 * kk, 32 * tiles.vt), v1 = col_op(sm.g + trl, R, 16 * kk, 32 * tiles.vt);
#pragma unroll
        for (int u = 0; u < TPW; ++u) {
          const bf16x8 f0 = col_op(sm.fk + trl, R, 16 * kk, 32 * (tiles.ft0 + u));
          const bf16x8 f1 = col_op(sm.fq + trl, R, 16 * kk, 32 * (tiles.ft0 + u));
          sacc[u] = mfma32(v0, f0, sacc[u]);
          sacc[u] = mfma32(v1, f1, sacc[u]);
          tiles.pick(z0[u], kk, f0);
          tiles.pick(z1[u], kk, f1);
        }
      }
#pragma unroll
      for (int u = 0; u < TPW; ++u) zs[u] = tiles.sum(z1[u], tiles.sum(z0[u], 0.f));
      tiles.put(sm.zpart, zs, ln, lh);
      lds_barrier();
      if (tid < D) {
        float zz = sm.z[tid];
#pragma unroll
        for (int pz = 0; pz < MT; ++pz) zz += sm.zpart[pz][tid];
        sm.z[tid] = zz;
      }
    }
    if (n0 >= cb) tiles.copy(sm.st, sacc, ln, lh);   // the next round scans: it reads the operand copy of the carried sum
  }

  load_chunk(n0);
  map_chunk(n0);
  stage_chunk(n0);
  if (n0 + 1 < ce) load_chunk(n0 + 1);
  lds_barrier();

  // The 64 x 64 products are three 32 x 32 tiles on or below the diagonal, one per wave 0..2: tokens 32*it.., 32*jt..
  const bool has_tile = wave < 3;
  const int it = wave > 0, jt = wave > 1;
  const int ot = wave % MT, it2 = wave / MT;            // output tile of the 64 x d products

  for (int n = n0; n < ce; ++n) {
    const int t0 = n * CH;
    const bool full = n >= cb;   // uniform over the workgroup
    f32x16 traw, racc;
    float inv = 1.f, ci = 0.f;   // 1 / den and c of token 32*it2 + ln
    if (full) {
    // ---- (a) S and T = dO v^T of a tile (a lane owns one token i, registers are tokens j), their sums over j; the tile
    //      (feature block ot, token block it2) of r = A dO with its part of phi(q).r and phi(q).Z ----
    if (has_tile) {
      f32x16 s;
#pragma unroll
      for (int r = 0; r < 16; ++r) { s[r] = 0.f; traw[r] = 0.f; }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        s = mfma32(row_op(sm.fk, R, 32 * jt, ks, ln, lh), row_op(sm.fq, R, 32 * it, ks, ln, lh), s);
        traw = mfma32(row_op(sm.v, R, 32 * jt, ks, ln, lh), row_op(sm.g, R, 32 * it, ks, ln, lh), traw);
      }
      float ss = 0.f, st = 0.f;
      const int top = (it == jt ? ln : CH) - 4 * lh;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        // T is masked as well: a later token's product may be infinite
        const bool seen = 8 * (r / 4) + r % 4 <= top;
        const float x = seen ? s[r] : 0.f;
        ss += x;
        st = fmaf(x, seen ? traw[r] : 0.f, st);
      }
      ss = sum_over_halves(ss);
      st = sum_over_halves(st);
      if (lh == 0) {
        sm.part[0][wave][ln] = ss;
        sm.part[1][wave][ln] = st;
      }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) racc[r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      racc = mfma32(row_op(sm.st, R, 32 * ot, ks, ln, lh), row_op(sm.g, R, 32 * it2, ks, ln, lh), racc);
    {
      const int i = 32 * it2 + ln;
      float qr = 0.f, qz = 0.f;
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const int f0 = 32 * ot + 8 * g4 + 4 * lh;
        const float4 z4 = *reinterpret_cast<const float4*>(&sm.z[f0]);
        float f[4];
        get4(&sm.fq[i * R + f0], f);
        qz = fmaf(f[0], z4.x, fmaf(f[1], z4.y, fmaf(f[2], z4.z, fmaf(f[3], z4.w, qz))));
#pragma unroll
        for (int e = 0; e < 4; ++e) qr = fmaf(f[e], racc[4 * g4 + e], qr);
      }
      qr = sum_over_halves(qr);
      qz = sum_over_halves(qz);
      if (lh == 0) {
        sm.red[0][ot][i] = qr;
        sm.red[1][ot][i] = qz;
      }
    }
    lds_barrier();

    // ---- (b) den and c; the T' tile ----
    auto den_and_c = [&](int tb, float& inv_out, float& c_out) {   // of token 32*tb + ln
      const int i = 32 * tb + ln;
      float qr = 0.f, qz = 0.f;
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        qr += sm.red[0][m][i];
        qz += sm.red[1][m][i];
      }
      qz += tb == 0 ? sm.part[0][0][ln] : sm.part[0][1][ln] + sm.part[0][2][ln];
      qr += tb == 0 ? sm.part[1][0][ln] : sm.part[1][1][ln] + sm.part[1][2][ln];
      const float den = t0 + i < N ? qz + a.eps : 1.f;   // rows past the end: dO is zero
      inv_out = 1.f / den;
      c_out = qr * inv_out * inv_out;
      return den;
    };
    const float den = den_and_c(it2, inv, ci);
    if (ot == 0 && lh == 0 && t0 + 32 * it2 + ln < N)
      *reinterpret_cast<float2*>(&hc.ws[2 * (int64_t)(t0 + 32 * it2 + ln)]) = make_float2(den, ci);
    if (has_tile) {
      float tinv, tc;
      den_and_c(it, tinv, tc);
      const int i = 32 * it + ln, top = (it == jt ? ln : CH) - 4 * lh;
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        float x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = 8 * g4 + e <= top ? fmaf(traw[4 * g4 + e], tinv, -tc) : 0.f;
        put4_split(&sm.tp[i * SR + 32 * jt + 8 * g4 + 4 * lh], &sm.tl[i * SR + 32 * jt + 8 * g4 + 4 * lh],
                   x[0], x[1], x[2], x[3]);
      }
    }
    }  // full

    // ---- (c) the carried sums: nothing here waits for T', so the waves without a tile go ahead ----
    float zs[TPW];
    typename SumTiles<D>::Picked fz[TPW];
#pragma unroll
    for (int kk = 0; kk < CH / 16; ++kk) {
      const bf16x8 vop = col_op(sm.v + trl, R, 16 * kk, 32 * tiles.vt);
#pragma unroll
      for (int u = 0; u < TPW; ++u) {
        const bf16x8 fop = col_op(sm.fk + trl, R, 16 * kk, 32 * (tiles.ft0 + u));
        sacc[u] = mfma32(vop, fop, sacc[u]);
        tiles.pick(fz[u], kk, fop);
      }
    }
#pragma unroll
    for (int u = 0; u < TPW; ++u) zs[u] = tiles.sum(fz[u], 0.f);
    tiles.put(sm.zpart, zs, ln, lh);
    lds_barrier();

    // ---- (d) dfq^T tile (feature block ot, token block it2) = r / den - c Z + T' fk ----
    if (full) {
      f32x16 dacc;
#pragma unroll
      for (int r = 0; r < 16; ++r) dacc[r] = 0.f;
#pragma unroll
      for (int kk = 0; kk < CH / 16; ++kk)
        if (16 * kk < 32 || it2 > 0) {   // tokens 0..31 see no others
          const bf16x8 kop = col_op(sm.fk + trl, R, 16 * kk, 32 * ot);
          dacc = mfma32(kop, row_op(sm.tp, SR, 32 * it2, kk, ln, lh), dacc);
          dacc = mfma32(kop, row_op(sm.tl, SR, 32 * it2, kk, ln, lh), dacc);
        }
      const int i = 32 * it2 + ln;
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const int f0 = 32 * ot + 8 * g4 + 4 * lh;
        const float4 z4 = *reinterpret_cast<const float4*>(&sm.z[f0]);
        const float zv[4] = {z4.x, z4.y, z4.z, z4.w};
        uint16_t* fp = &sm.fq[i * R + f0];   // this wave's own corner of the tile: dq replaces phi(q)
        float fv[4], x[4];
        get4(fp, fv);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          x[e] = (fmaf(racc[4 * g4 + e], inv, dacc[4 * g4 + e]) - ci * zv[e]) * slope_of<ELU1>(fv[e]);
        put4(fp, x[0], x[1], x[2], x[3]);
      }
    }
    lds_barrier();

    // ---- (e) hand the sums to the next chunk; dq rows out; next chunk in ----
    if (n + 1 >= cb) tiles.copy(sm.st, sacc, ln, lh);   // light rounds do not read the operand copy
    if (tid < D) {
      float zz = sm.z[tid];
#pragma unroll
      for (int pz = 0; pz < MT; ++pz) zz += sm.zpart[pz][tid];
      sm.z[tid] = zz;
    }
    if (full) {
#pragma unroll
      for (int i = 0; i < PCS; ++i) {
        const int p = tid + i * NT, row = p / C::C8, col = 8 * (p % C::C8);
        if (t0 + row < N)
          *reinterpret_cast<u32x4*>(dqp + (int64_t)(t0 + row) * a.q.sn + col) =
              *reinterpret_cast<const u32x4*>(&sm.fq[row * R + col]);
      }
    }
    if (n + 1 < ce) {
      map_chunk(n + 1);
      stage_chunk(n + 1);   // the same thread overwrites the pieces it has just read
    }
    if (n + 2 < ce) load_chunk(n + 2);
    lds_barrier();
  }
}

// ---------------------------------------------------------------------------------------
// reverse scan: dk, dv from (den_i, c_i) of the workspace
// ---------------------------------------------------------------------------------------
template <int D, bool ELU1>
__device__ __forceinline__ void scan_kv(const BwdArgs& a, int h, int b, int seg, unsigned char* smem_raw) {
  using C = LbCfg<D>;
  constexpr int MT = C::MT, KS = C::KS, NW = C::NW, NT = C::NT, R = C::R, TPW = C::TPW, PCS = C::PCS;
  LbSmemKv<D>& sm = *reinterpret_cast<LbSmemKv<D>*>(smem_raw);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, ln = lane & 31, lh = lane >> 5;
  const HeadCtx<D> hc = head_ctx<D>(a, b, h);
  uint16_t* dkp = reinterpret_cast<uint16_t*>(a.dk) + b * a.k.sb + h * a.k.sh;
  uint16_t* dvp = reinterpret_cast<uint16_t*>(a.dv) + b * a.v.sb + h * a.v.sh;
  const int N = a.N, nchunks = (N + CH - 1) / CH;
  // this workgroup writes the chunks [cb, ce) of its head; the chunks behind them are only summed
  const int cb = nchunks - a.lin_bounds[seg + 1], ce = nchunks - a.lin_bounds[seg];
  if (cb >= ce) return;
  const int trl = lds_operand_tr_lane_offset(R, lane) + 8 * lh * R;

  u32x4 rq[PCS], rk[PCS], rv[PCS], rdo[PCS];
  float2 rstat = {1.f, 0.f};
  auto load_chunk = [&](int n) {
    const bool full = n < ce;   // uniform
#pragma unroll
    for (int i = 0; i < PCS; ++i) {
      const int p = tid + i * NT, row = p / C::C8, col = 8 * (p % C::C8);
      const int64_t tok = min(n * CH + row, N - 1);
      rq[i] = *reinterpret_cast<const u32x4*>(hc.q + tok * a.q.sn + col);
      rdo[i] = *reinterpret_cast<const u32x4*>(hc.dout + tok * a.dout.sn + col);
      if (full) {
        rk[i] = *reinterpret_cast<const u32x4*>(hc.k + tok * a.k.sn + col);
        rv[i] = *reinterpret_cast<const u32x4*>(hc.v + tok * a.v.sn + col);
      }
    }
    if (tid < CH) rstat = *reinterpret_cast<const float2*>(&hc.ws[2 * (int64_t)min(n * CH + tid, N - 1)]);
  };
  auto map_chunk = [&](int n) {
    const bool full = n < ce;
#pragma unroll
    for (int i = 0; i < PCS; ++i) {
      rq[i] = map8<ELU1>(rq[i]);
      if (full) rk[i] = map8<ELU1>(rk[i]);
    }
  };
  auto stage_chunk = [&](int n) {
    const bool full = n < ce;
#pragma unroll
    for (int i = 0; i < PCS; ++i) {
      const int p = tid + i * NT, row = p / C::C8, col = 8 * (p % C::C8);
      const bool valid = n * CH + row < N;
      *reinterpret_cast<u32x4*>(&sm.fq[row * R + col]) = valid ? rq[i] : kZero4;
      *reinterpret_cast<u32x4*>(&sm.g[row * R + col]) = valid ? rdo[i] : kZero4;
      if (full) {
        *reinterpret_cast<u32x4*>(&sm.fk[row * R + col]) = valid ? rk[i] : kZero4;
        *reinterpret_cast<u32x4*>(&sm.v[row * R + col]) = valid ? rv[i] : kZero4;
      }
    }
    if (tid < CH) {
      const bool valid = n * CH + tid < N;
      sm.cc[tid] = valid ? rstat.y : 0.f;
      sm.den[tid] = valid ? 1.f / rstat.x : 1.f;
    }
  };

  const SumTiles<D> tiles(wave);   // B^T
  f32x16 sacc[TPW];
#pragma unroll
  for (int u = 0; u < TPW; ++u)
#pragma unroll
    for (int r = 0; r < 16; ++r) sacc[u][r] = 0.f;
  for (int i = tid; i < D * R / 2; i += NT) reinterpret_cast<uint32_t*>(sm.st)[i] = 0u;
  if (tid < D) sm.z[tid] = 0.f;

  // Light rounds, two chunks at a time (the chunks behind the segment only feed the carried
  // sums): phi(q), g and c of chunk n go to the fq / g tiles and cc, those of chunk n - 1 to the
  // fk / v tiles and dz (and travel in the k / v staging registers).
  float rden[PCS], rden2[PCS];
  float2 rstat2 = {1.f, 0.f};
  auto load_pair = [&](int n) {
#pragma unroll
    for (int i = 0; i < PCS; ++i) {
      const int p = tid + i * NT, row = p / C::C8, col = 8 * (p % C::C8);
      const int64_t t0 = min(n * CH + row, N - 1), t1 = (n - 1) * CH + row;
      rq[i] = *reinterpret_cast<const u32x4*>(hc.q + t0 * a.q.sn + col);
      rdo[i] = *reinterpret_cast<const u32x4*>(hc.dout + t0 * a.dout.sn + col);
      rden[i] = hc.ws[2 * t0];
      rk[i] = *reinterpret_cast<const u32x4*>(hc.q + t1 * a.q.sn + col);
      rv[i] = *reinterpret_cast<const u32x4*>(hc.dout + t1 * a.dout.sn + col);
      rden2[i] = hc.ws[2 * t1];
    }
    if (tid < CH) {
      rstat = *reinterpret_cast<const float2*>(&hc.ws[2 * (int64_t)min(n * CH + tid, N - 1)]);
      rstat2 = *reinterpret_cast<const float2*>(&hc.ws[2 * (int64_t)((n - 1) * CH + tid)]);
    }
  };
  int n1 = nchunks - 1;   // first chunk of the round-by-round loop below
  if (nchunks - ce >= 2) {
    load_pair(n1);
    for (; n1 - 1 >= ce; n1 -= 2) {
#pragma unroll
      for (int i = 0; i < PCS; ++i) {
        const int p = tid + i * NT, row = p / C::C8, col = 8 * (p % C::C8);
        const bool valid = n1 * CH + row < N;   // only the head's last chunk can be ragged
        *reinterpret_cast<u32x4*>(&sm.fq[row * R + col]) = valid ? map8<ELU1>(rq[i]) : kZero4;
        *reinterpret_cast<u32x4*>(&sm.g[row * R + col]) = valid ? scale8(rdo[i], 1.f / rden[i]) : kZero4;
        *reinterpret_cast<u32x4*>(&sm.fk[row * R + col]) = map8<ELU1>(rk[i]);
        *reinterpret_cast<u32x4*>(&sm.v[row * R + col]) = scale8(rv[i], 1.f / rden2[i]);
      }
      if (tid < CH) {
        sm.cc[tid] = (n1 * CH + tid < N) ? rstat.y : 0.f;
        sm.dz[tid] = rstat2.y;
      }
      if (n1 - 3 >= ce) load_pair(n1 - 2);
      lds_barrier();
      float zs[TPW];
      typename SumTiles<D>::Picked z0[TPW], z1[TPW];
#pragma unroll
      for (int kk = 0; kk < CH / 16; ++kk) {
        const bf16x8 g0 = col_op(sm.g + trl, R, 16 * kk, 32 * tiles.vt), g1 = col_op(sm.v + trl, R, 16 * kk, 32 * tiles.vt);
#pragma unroll
        for (int u = 0; u < TPW; ++u) {
          const bf16x8 f0 = col_op(sm.fq + trl, R, 16 * kk, 32 * (tiles.ft0 + u));
          const bf16x8 f1 = col_op(sm.fk + trl, R, 16 * kk, 32 * (tiles.ft0 + u));
          sacc[u] = mfma32(g0, f0, sacc[u]);
          sacc[u] = mfma32(g1, f1, sacc[u]);
          tiles.pick(z0[u], kk, f0);
          tiles.pick(z1[u], kk, f1);
        }
      }
#pragma unroll
      for (int u = 0; u < TPW; ++u) zs[u] = tiles.sum(z1[u], sm.dz, lh, tiles.sum(z0[u], sm.cc, lh, 0.f));
      tiles.put(sm.zpart, zs, ln, lh);
      lds_barrier();
      if (tid < D) {
        float yy = sm.z[tid];
#pragma unroll
        for (int pz = 0; pz < MT; ++pz) yy += sm.zpart[pz][tid];
        sm.z[tid] = yy;
      }
    }
    if (n1 < ce) tiles.copy(sm.st, sacc, ln, lh);   // the next round scans: it reads the operand copy of the carried sum
  }

  load_chunk(n1);
  map_chunk(n1);
  stage_chunk(n1);
  if (n1 - 1 >= cb) load_chunk(n1 - 1);
  lds_barrier();

  const int ti = wave & 3, it = ti & 1, jt = ti >> 1;   // here rows are i, columns j (a lane owns a key j)
  const bool none = it < jt;   // queries 0..31 see no keys 32..63: that tile is neither made nor read
  const bool do_s = !none && (NW == 4 || wave < 4), do_t = !none && (NW == 4 || wave >= 4);
  const int ot = wave % MT, jt2 = wave / MT;

  for (int n = n1; n >= cb; --n) {
    const int t0 = n * CH;
    const bool full = n < ce;   // uniform over the workgroup
    // ---- (a) S / den and T' tiles, stored transposed ([j][i]) ----
    if (full && do_s) {
      f32x16 s;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        s = mfma32(row_op(sm.fq, R, 32 * it, ks, ln, lh), row_op(sm.fk, R, 32 * jt, ks, ln, lh), s);
      const int j = 32 * jt + ln;
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const float4 r4 = *reinterpret_cast<const float4*>(&sm.den[32 * it + 8 * g4 + 4 * lh]);
        const float rv4[4] = {r4.x, r4.y, r4.z, r4.w};
        float x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int i = 32 * it + 8 * g4 + 4 * lh + e;
          x[e] = j <= i ? s[4 * g4 + e] * rv4[e] : 0.f;
        }
        put4(&sm.sm[j * SR + 32 * it + 8 * g4 + 4 * lh], x[0], x[1], x[2], x[3]);
      }
    }
    if (full && do_t) {
      f32x16 tr;
#pragma unroll
      for (int r = 0; r < 16; ++r) tr[r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        tr = mfma32(row_op(sm.g, R, 32 * it, ks, ln, lh), row_op(sm.v, R, 32 * jt, ks, ln, lh), tr);
      const int j = 32 * jt + ln;
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const float4 c4 = *reinterpret_cast<const float4*>(&sm.cc[32 * it + 8 * g4 + 4 * lh]);
        const float4 r4 = *reinterpret_cast<const float4*>(&sm.den[32 * it + 8 * g4 + 4 * lh]);
        const float cv[4] = {c4.x, c4.y, c4.z, c4.w}, rv4[4] = {r4.x, r4.y, r4.z, r4.w};
        float x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int i = 32 * it + 8 * g4 + 4 * lh + e;
          x[e] = j <= i ? fmaf(tr[4 * g4 + e], rv4[e], -cv[e]) : 0.f;
        }
        put4_split(&sm.tp[j * SR + 32 * it + 8 * g4 + 4 * lh], &sm.tl[j * SR + 32 * it + 8 * g4 + 4 * lh],
                   x[0], x[1], x[2], x[3]);
      }
    }
    lds_barrier();

    // ---- (b) dfk^T tile (feature block ot, key block jt2), dv^T tile (value block ot), B^T ----
    f32x16 kacc, vacc;
#pragma unroll
    for (int r = 0; r < 16; ++r) { kacc[r] = 0.f; vacc[r] = 0.f; }
    if (full) {
#pragma unroll
    for (int kk = 0; kk < CH / 16; ++kk)
      if (16 * kk >= 32 || jt2 == 0) {
        const bf16x8 qop = col_op(sm.fq + trl, R, 16 * kk, 32 * ot);
        kacc = mfma32(qop, row_op(sm.tp, SR, 32 * jt2, kk, ln, lh), kacc);
        kacc = mfma32(qop, row_op(sm.tl, SR, 32 * jt2, kk, ln, lh), kacc);
      }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      kacc = mfma32(row_op(sm.st, R, 32 * ot, ks, ln, lh), row_op(sm.v, R, 32 * jt2, ks, ln, lh), kacc);
#pragma unroll
    for (int kk = 0; kk < CH / 16; ++kk)
      if (16 * kk >= 32 || jt2 == 0)
        vacc = mfma32(col_op(sm.g + trl, R, 16 * kk, 32 * ot), row_op(sm.sm, SR, 32 * jt2, kk, ln, lh), vacc);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      vacc = mfma32(col_op(sm.st + trl, R, 16 * ks, 32 * ot), row_op(sm.fk, R, 32 * jt2, ks, ln, lh), vacc);
    }  // full
    float zs[TPW];
    typename SumTiles<D>::Picked fz[TPW];
#pragma unroll
    for (int kk = 0; kk < CH / 16; ++kk) {
      const bf16x8 gop = scaled8(col_op(sm.g + trl, R, 16 * kk, 32 * tiles.vt), sm.den + 16 * kk + 8 * lh);
#pragma unroll
      for (int u = 0; u < TPW; ++u) {
        const bf16x8 fop = col_op(sm.fq + trl, R, 16 * kk, 32 * (tiles.ft0 + u));
        sacc[u] = mfma32(gop, fop, sacc[u]);
        tiles.pick(fz[u], kk, fop);
      }
    }
#pragma unroll
    for (int u = 0; u < TPW; ++u) zs[u] = tiles.sum(fz[u], sm.cc, lh, 0.f);
    tiles.put(sm.zpart, zs, ln, lh);
    lds_barrier();   // every read of the phi(k) and v tiles is done

    // ---- (c) dk replaces phi(k), dv replaces v ----
    if (full) {
      const int j = 32 * jt2 + ln;
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const int c0 = 32 * ot + 8 * g4 + 4 * lh;
        const float4 y4 = *reinterpret_cast<const float4*>(&sm.z[c0]);
        uint16_t* fp = &sm.fk[j * R + c0];
        float fv[4];
        get4(fp, fv);
        put4(fp, (kacc[4 * g4 + 0] - y4.x) * slope_of<ELU1>(fv[0]), (kacc[4 * g4 + 1] - y4.y) * slope_of<ELU1>(fv[1]),
             (kacc[4 * g4 + 2] - y4.z) * slope_of<ELU1>(fv[2]), (kacc[4 * g4 + 3] - y4.w) * slope_of<ELU1>(fv[3]));
        put4(&sm.v[j * R + c0], vacc[4 * g4 + 0], vacc[4 * g4 + 1], vacc[4 * g4 + 2], vacc[4 * g4 + 3]);
      }
    }
    lds_barrier();

    // ---- (d) hand the sums on; dk, dv rows out; next (earlier) chunk in ----
    if (n - 1 < ce) tiles.copy(sm.st, sacc, ln, lh);   // light rounds do not read the operand copy
    if (tid < D) {
      float yy = sm.z[tid];
#pragma unroll
      for (int pz = 0; pz < MT; ++pz) yy += sm.zpart[pz][tid];
      sm.z[tid] = yy;
    }
    if (full) {
#pragma unroll
      for (int i = 0; i < PCS; ++i) {
        const int p = tid + i * NT, row = p / C::C8, col = 8 * (p % C::C8);
        if (t0 + row < N) {
          *reinterpret_cast<u32x4*>(dkp + (int64_t)(t0 + row) * a.k.sn + col) =
              *reinterpret_cast<const u32x4*>(&sm.fk[row * R + col]);
          *reinterpret_cast<u32x4*>(dvp + (int64_t)(t0 + row) * a.v.sn + col) =
              *reinterpret_cast<const u32x4*>(&sm.v[row * R + col]);
        }
      }
    }
    if (n - 1 >= cb) {
      map_chunk(n - 1);
      stage_chunk(n - 1);
    }
    if (n - 2 >= cb) load_chunk(n - 2);
    lds_barrier();
  }
}

// ---- launches --------------------------------------------------------------------------------------
// A scan, and behind it in the same launch passes over the windowed heads' band: blocks [0, linear) scan,
// the `rows` blocks from the next multiple of 8 on (the XCDs keep their runs) are dq's in the forward scan's
// launch and dk's in the reverse scan's, and behind those in the forward scan's come dv's.
// A scan is one workgroup per compute unit and rarely as many of them as there are units, the band's passes are
// many short workgroups: they run on the units the scans leave, and behind the scans that end first.  A band
// workgroup takes the scans' eight waves (256 resident rows, the same bits as 128).  Measured, all passes apart
// and together (us): 4 x (6 + 26 heads) x 8192 tokens, window 256: 1155 and 1091; 8 x (6 + 42) x 2048, 128: 888
// and 796; 1 x (28 + 4) x 4096, 256: 460 and 332; 16 x (30 + 10) x 1024, 128: 723 and 706; 1 x (1 + 1) x 300,
// 64: 98 and 70.  Two separate bands of 128 rows in a workgroup: the same times, and 726 for the fourth.
// A launch without a band has a kernel without its code, and (heads, batch, segments) for a grid: with the band's
// branches in it the two scans of 32 heads x 1000 tokens took 83.2 us in place of 81.7, of 8 x 512 63.4 in place of
// 62.0 (the same on long calls, where the scans' chunks are everything).
template <int D, bool ELU1, bool REVERSE, bool BAND>
__global__ __launch_bounds__(LbCfg<D>::NT, 1) void linear_bwd_scan_kernel(BwdArgs a, int linear, int rows) {
  constexpr int NT = LbCfg<D>::NT;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  const int H1 = a.H - a.H0, block = blockIdx.x;
  int head = block, b = blockIdx.y, seg = blockIdx.z;
  if constexpr (BAND) {
    const int first = (linear + 7) & ~7, second = first + ((rows + 7) & ~7);
    if (block >= first) {
      if (block < first + rows) windowed_band<D, REVERSE ? kDk : kDq, NT>(a, block - first, smem_raw);
      else if (!REVERSE && block >= second) windowed_band<D, kDv, NT>(a, block - second, smem_raw);
      return;
    }
    if (block >= linear) return;
    head = block % H1;
    b = block / H1 % a.B;
    seg = block / (H1 * a.B);
  }
  if constexpr (REVERSE) scan_kv<D, ELU1>(a, a.H0 + head, b, seg, smem_raw);
  else scan_q<D, ELU1>(a, a.H0 + head, b, seg, smem_raw);
}

template <int D, bool ELU1, bool BAND> hipError_t launch_lin_bwd_t(const BwdArgs& a, hipStream_t s) {
  constexpr int NT = LbCfg<D>::NT, BR = band_rows(NT);
  static_assert(!BAND || (sizeof(BandSmem<D>) <= sizeof(LbSmem<D>) && sizeof(BandSmem<D>) <= sizeof(LbSmemKv<D>)),
                "the band's tiles fit the scans' LDS");
  const int linear = (a.H - a.H0) * a.B * a.lin_segments, first = (linear + 7) & ~7;
  const int rows = BAND ? (a.N + BR - 1) / BR * a.H0 * a.B : 0;
  hipError_t e = hipSuccess;
  auto launch = [&](auto kern, size_t smem, int blocks) {
    if (e != hipSuccess) return;
    e = allow_lds(kern, smem);
    if (e == hipSuccess) kern<<<BAND ? dim3(blocks) : dim3(a.H - a.H0, a.B, a.lin_segments), dim3(NT), smem, s>>>(a, linear, rows);
  };
  launch(linear_bwd_scan_kernel<D, ELU1, false, BAND>, sizeof(LbSmem<D>), first + ((rows + 7) & ~7) + rows);
  launch(linear_bwd_scan_kernel<D, ELU1, true, BAND>, sizeof(LbSmemKv<D>), first + rows);
  return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace

// Linear heads [H0, H) of a bf16 call; the workspace receives (den_i, c_i) per token.
hipError_t launch_linear_backward_mfma(const BwdArgs& args, bool with_windowed, hipStream_t s) {
  if (args.H - args.H0 <= 0 || args.N <= 0 || args.B <= 0) return hipSuccess;
  // A head is one sequential scan.  With fewer heads than compute units each head is cut into
  // segments, one workgroup per segment: it first sums the chunks in front of (behind) its
  // segment in light rounds, then scans the segment.
  BwdArgs a = args;
  const int heads = (a.H - a.H0) * a.B, nchunks = (a.N + CH - 1) / CH;
  a.lin_segments = std::max(1, std::min(std::min(4, device_compute_units() / heads), nchunks / 4));
  // A chunk of a light round costs about a quarter of a chunk of a full round (measured: the
  // step is flat between 0.7 and 0.8 below), and segment s runs the light rounds of everything in
  // front of it: lengths in the ratio 0.75^s finish together.  The reverse scan uses the same cut
  // mirrored.
  {
    double wsum = 0.0, w = 1.0;
    for (int sgm = 0; sgm < a.lin_segments; ++sgm, w *= 0.75) wsum += w;
    double acc = 0.0;
    w = 1.0;
    a.lin_bounds[0] = 0;
    for (int sgm = 1; sgm <= a.lin_segments; ++sgm, w *= 0.75) {
      acc += w;
      a.lin_bounds[sgm] = sgm == a.lin_segments ? nchunks : std::min(nchunks, (int)(nchunks * acc / wsum + 0.5));
    }
  }
  const bool elu1 = a.phi == 0;
  if (a.d == 64) return elu1 ? launch_lin_bwd_t<64, true, false>(a, s) : launch_lin_bwd_t<64, false, false>(a, s);
  if (with_windowed) return elu1 ? launch_lin_bwd_t<128, true, true>(a, s) : launch_lin_bwd_t<128, false, true>(a, s);
  return elu1 ? launch_lin_bwd_t<128, true, false>(a, s) : launch_lin_bwd_t<128, false, false>(a, s);
}

}  // namespace gformer
