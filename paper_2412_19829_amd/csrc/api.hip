// C ABI of the GFormer attention library: argument validation, launch planning, dispatch.
// Everything up to the first launch is plain host code and can be exercised without a GPU.
#include "../../include/gformer.h"

#include <string.h>

#include <algorithm>
#include <mutex>

#include "common.hpp"

#include <atomic>

namespace gformer {

int mfma_linear_threads(int d, int query_halves) { return d == 128 ? 512 : 256 * query_halves; }

// Compute units of the current device, asked once per device; a process without a device (the
// planner is host arithmetic and is also called there) plans for an MI355X.
int device_compute_units() {
  constexpr int kDefault = 256, kSlots = 64;
  static std::atomic<int> cached[kSlots];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kSlots) {
    (void)hipGetLastError();
    return kDefault;
  }
  int n = cached[dev].load(std::memory_order_relaxed);
  if (n > 0) return n;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) {
    (void)hipGetLastError();
    return kDefault;
  }
  cached[dev].store(n, std::memory_order_relaxed);
  return n;
}

namespace {

struct Resolved {
  gformer_plan plan;
  int64_t qs[3], ks[3], vs[3], os[3];
  int cph, vcph, piece_chunks, state_sub, query_halves;
  bool stream;   // MFMA path: the windowed heads go to the streaming kernel
  bool general_chunk;  // MFMA path, causal: the linear read-out goes to the general-chunk kernel
  bool f32;            // single precision on the matrix cores
  int f32_seg_len, f32_nseg;
  uint64_t needed;     // workspace of this cut; plan.workspace_bytes, which is reported, serves every form of the shape
};

// Single-precision calls run on the matrix cores (fp32 operands and accumulation) unless the caller
// asks for the plain-FMA kernels, or has more rows or heads than one grid of the former can name.
bool f32_matrix(const gformer_params* p, int B, int H, int N) {
  return p->dtype == GF_F32 && p->impl == GF_IMPL_AUTO && (int64_t)B * H * ((N + 15) / 16) < kF32MaxRows / 16;
}

// One side stream and a fork/join event pair per device, created on first use and kept for the
// life of the process.  Default priority on purpose.
constexpr int kMaxDevices = 64;
struct SideStream {
  bool ready = false;
  hipStream_t stream = nullptr;
  hipEvent_t fork = nullptr, join = nullptr;
};
SideStream g_side[kMaxDevices];
std::mutex g_enqueue_mutex;

// The device a call works on: the current one, which must also be the device of the caller's
// stream when that is not the null stream (kernels launched on a stream run on the stream's
// device, while per-device state below is looked up by the current one).
hipError_t call_device(hipStream_t s, int* dev) {
  hipError_t e = hipGetDevice(dev);
  if (e != hipSuccess) return e;
  if (s != nullptr) {
    int sdev = -1;
    // a stream under capture may refuse the query; the device check is then skipped
    if (hipStreamGetDevice(s, &sdev) == hipSuccess) {
      if (sdev != *dev) return hipErrorInvalidDevice;
    } else {
      (void)hipGetLastError();
    }
  }
  if (*dev < 0 || *dev >= kMaxDevices) return hipErrorInvalidDevice;
  return hipSuccess;
}

hipError_t side_stream_for_current_device(hipStream_t caller, SideStream** out) {
  int dev = 0;
  hipError_t e = call_device(caller, &dev);
  if (e != hipSuccess) return e;
  SideStream& s = g_side[dev];
  if (!s.ready) {
    if ((e = hipStreamCreateWithFlags(&s.stream, hipStreamNonBlocking)) != hipSuccess) return e;
    if ((e = hipEventCreateWithFlags(&s.fork, hipEventDisableTiming)) != hipSuccess) return e;
    if ((e = hipEventCreateWithFlags(&s.join, hipEventDisableTiming)) != hipSuccess) return e;
    s.ready = true;
  }
  *out = &s;
  return hipSuccess;
}

// Scratch of the entry point that allocates nothing: the carried linear-attention states live in
// this file-scope device array instead of a caller's workspace.  Every device the library runs
// on holds its own copy, at its own address, from the moment the code object is loaded until the
// process ends.  In host code the array's name is only a handle for hipGetSymbolAddress; the
// address that kernels receive is looked up once per device, with that device current.
constexpr size_t kScratchBytes = GFORMER_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
std::atomic<void*> g_scratch_ptr[kMaxDevices];

hipError_t scratch_for_current_device(hipStream_t caller, void** out) {
  int dev = 0;
  hipError_t e = call_device(caller, &dev);
  if (e != hipSuccess) return e;
  void* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (!ptr) {
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev].store(ptr, std::memory_order_release);
  }
  *out = ptr;
  return hipSuccess;
}

constexpr int64_t kMaxRowStride = 1 << 20;  // elements

bool strides_all_zero(const int64_t* s) { return s[0] == 0 && s[1] == 0 && s[2] == 0; }

void dense_strides(int64_t* s, int H, int N, int d) {
  s[0] = (int64_t)H * N * d;
  s[1] = (int64_t)N * d;
  s[2] = d;
}

gf_status check_strides(const int64_t* in, int64_t* out, int H, int N, int d) {
  if (strides_all_zero(in)) {
    dense_strides(out, H, N, d);
    return GF_OK;
  }
  for (int i = 0; i < 3; ++i) {
    if (in[i] < 0 || (in[i] % 8) != 0) return GF_ERR_INVALID_ARG;
    out[i] = in[i];
  }
  if (N > 1 && in[2] < d) return GF_ERR_INVALID_ARG;  // rows would overlap
  if (in[2] > kMaxRowStride) return GF_ERR_UNSUPPORTED;  // kernels keep in-chunk offsets in 32 bits
  return GF_OK;
}


// Chunks per piece when every linear head is cut into the same whole number of pieces (one
// workgroup per piece, at most one per compute unit, pieces of 8 chunks or more), or 0 when that
// would leave more than a fifth of the compute units without a piece.
long aligned_piece(long heads_lin, long cph, long kComputeUnits) {
  if (heads_lin <= 0 || cph <= 0) return 0;
  long k = kComputeUnits / heads_lin;
  if (k > cph / 8) k = cph / 8;
  if (k < 1) return 0;
  const long piece = (cph + k - 1) / k;
  const long per_head = (cph + piece - 1) / piece;
  if (heads_lin * per_head * 5 < (long)kComputeUnits * 4) return 0;
  return piece;
}

// Chunks per piece of a small call, or 0 where this rule does not apply: no whole-number cut fills the
// chip, and pieces of eight chunks would leave more than three of eight compute units idle or every
// piece can be a whole short head.  Such a call takes as long as one
// piece: its chunks one after another, plus the sums it adds up first.  Uniform segments per head,
// shorter than eight chunks, trade the former for the latter.  Whole layer, us, pieces of eight
// against these:  d = 64, linear heads x chunks:  10x8 18.2 / 13.0 (2 chunks a piece), 10x16 24.8 / 14.9
// (2), 10x32 26.0 / 20.5 (4), 10x64 34.7 / 28.8 (4), 26x16 25.5 / 17.4 (3), 52x16 26.7 / 22.4 (4), 100x10
// 26.9 / 21.1 (5), 300x5 27.9 / 18.1 (5: a whole head, no carried sums at all; 17.6 in the present build).  d = 128, where a sum is
// four times as large and a compute unit holds one piece: 10x8 33.0 / 30.6 (2), 10x16 42.8 / 38.1 (4),
// 10x64 61.8 / 55.1 (4), 26x32 60.9 / 54.8 (6), 52x10 47.8 / 40.4 (5).  Two-chunk pieces lose where they crowd the chip
// (the present build, pieces of two, three, four: 26x16 18.9, 17.8, 19.5; 52x16 25.6, 25.1, 21.0).  That a head gets no more
// than eight of them was drawn when the sums of more were added up more slowly (10x32 23.2 then); now they would be
// faster there too (10x18 15.3, 16.5, 18.7; 10x25 18.3, 17.7, 19.3; 10x32 19.1, 20.7, 20.5; 10x48 21.4, 22.0, 23.7).
long short_piece(long heads, long cph, long cus, int d) {
  if (cph < 4 || heads <= 0 || heads > 2 * cus) return 0;
  if (heads * cph > 5 * cus && (heads * 5 < 4 * cus || cph > 8)) return 0;
  if (d == 128) {
    if (cph > 64 || heads > cus) return 0;
    long k = cus * 5 / 8 / heads;
    if (k > (cph <= 8 ? cph / 2 : cph / 4)) k = cph <= 8 ? cph / 2 : cph / 4;
    if (k < 1) k = 1;
    return (cph + k - 1) / k;
  }
  long k = cus / heads;
  if (k > cph / 2) k = cph / 2;
  if (k < 1) k = 1;
  long piece = (cph + k - 1) / k;
  const long per = (cph + piece - 1) / piece;
  if (per > 8 && piece < 4) piece = 4;
  else if (piece < 3 && heads * per > cus / 2) piece = 3;
  return piece;
}

// d = 64: whether the read-out's workgroup splits a chunk's queries over twice the waves (MainCfg, linear_mfma.hip), which makes
// a chunk shorter and a carried sum, which every set of waves loads, dearer.  Figures are us, four waves and eight.  Four waves:
// * pieces of one chunk, and pieces of up to four that start from more sums than they have chunks.  1 x 12 x 1024 (2 chunks, 7
//   sums) 14.7 and 15.6, x 512 (2, 3) 12.0 and 12.3, x 2048 (4, 7) 19.7 and 20.3; but 4 x 12 x 512 (3, 2) 15.9 and 15.0,
//   1 x 8 x 686 (3, 3) 14.4 and 13.6, 1 x 12 x 4096 (4, 1: scanned) 24.7 and 23.5.  Over all keys, where a chunk is short, more
//   sums than half the chunks: 1 x 12 x 512 (1, 8) 11.9 and 14.5, 3 x 12 x 1951 (5, 7) 23.1 and 24.2, 4 x 12 x 2857 (9, 5) 27.4 and
//   28.3; but 5 x 8 x 4578 (12, 6) 33.6 and 34.0, 2 x 32 x 2326 (10, 4) 29.5 and 28.6.
// * more causal pieces than units: of four waves a unit holds two workgroups, of eight one, and the pieces take two rounds.
//   All heads linear: 257 x 320 16.6 and 19.2, 300 x 512 24.8 and 28.2, 384 x 400 22.1 and 25.2,
//   512 x 512 28.2 and 31.8, segments of 64 tokens 4 x 12 x 4096 77.7 and 94.0, of 512 1 x 48 x 4096 47.3 and 54.2 (256 x
//   400 16.2 and 14.6, 230 x 512 18.1 and 16.1).
// * over all keys, where a chunk is short: two to three pieces a unit (600 x 200 28.0 and 28.3; 384 x 577 35.3 and 34.7), and
//   features mapped beforehand, which leave nothing to hide (8 x 12 x 1000 19.0 and 19.5, 2 x 12 x 1325 15.7 and 18.2, but 3 x 8 x
//   31024 79.4 and 78.1; causal the staging still counts: 16 x 16 x 1024 30.4 and 26.3, 1 x 32 x 16384 87.6 and 79.1).
// With windowed heads the rule also says whose launch their query blocks share: the read-out's (four waves), which costs least
// where the layer is short, or the state pass's (eight).  The whole layer, heads as windowed + linear, window:
// * no state pass to share: four.  16 x (2 + 10) x 300, 64 13.2 and 17.5; 14 x (1 + 15) x 1089, 331 36.4 and 41.5.
// * pieces of two to four chunks: four, but for more workgroups of four waves than the chip holds.  1 x (2 + 10) x 512, 128 12.4
//   and 15.5; 18 x (3 + 5) x 364, 64 16.9 and 18.1; 1 x (1 + 7) x 5615, 256 25.3 and 27.0; 1 x (11 + 5) x 5484, 256 35.1 and 32.1.
//   Of five on: eight.  8 x (2 + 10) x 1024, 128 (6 chunks) 26.4 and 25.8; 3 x (1 + 11) x 2472, 38 (8) 35.8 and 32.9; 1 x (2 + 14)
//   x 16384, 128 (15) 56.0 and 49.4; 8 x (2 + 10) x 4096, 256 (22) 65.2 and 62.5; 4 x (1 + 31) x 16384, 64 (128) 284 and 258.
// * a query block's tiles a chain half as long again as a sum's chunks: four.  6 x (4 + 12) x 1241, 278 (7 tiles, 4 chunks) 32.4
//   and 34.0; mapped 2 x (1 + 31) x 1533, 274 (7, 4) 28.2 and 30.4.  Longer at all, where sums are few (five of eight units) and the
//   four-wave launch fits the chip: 3 x (1 + 31) x 613, 256, prefill (6, 5; 93 sums) 21.5 and 23.9; but 1 x (1 + 11) x 6288, 256 (6,
//   5; 209) 31.0 and 29.6.
// * pieces longer than a head, beside query blocks of fewer tiles than a sum has chunks that weigh more and with the pieces come to
//   nearly two a unit (19 to 10): four.  Few sums are left then, the query blocks run alone, and the read-out leaves most units idle
//   behind them.  29 x (12 + 4) x 188, 256 (44 pieces, 696 query blocks) 24.9 and 29.8; 20 x (24 + 8) x 136, 39 (60, 960) 24.6 and 29.1;
//   15 x (13 + 19) x 133, 256 (107, 390) 24.3 and 26.1; but 17 x (13 + 3) x 191, 64 (20, 442) 23.8 and 22.8; 22 x (17 + 15) x 624, 378
//   (more tiles) 76.5 and 71.5; 12 x (2 + 30) x 2578, 256 (lighter) 128.8 and 118.4.
// * sums of four chunks that with the query blocks take a second round (three a unit), where the four-wave launch takes no third (two a
//   unit): four where the query blocks are five times the weight, or the sums half as many again as the pieces.  11 x (7 + 1) x 1278, 128
//   (44 sums, 770 query blocks) 27.8 and 29.8; 6 x (8 + 8) x 1700, 28 (288, 672; 162 pieces) 33.7 and 37.7; 5 x (8 + 8) x 2267, 256 (300,
//   720; 180) 42.5 and 45.6; but 2 x (14 + 2) x 2850, 256 (44, 644) 33.5 and 30.8; 25 x (4 + 4) x 1009, 64 (200, 800; 200) 38.3 and 36.7.
// * mapped beforehand: eight for pieces of eight chunks on beside few tiles, two or less to five chunks.  Tiles a chunk, chunks
//   a piece: 8 x (2 + 10) x 1024, 128 (0.36, 6) 23.3 and 24.8; 9 x (2 + 6) x 5166, 256 (0.97, 21) 60.4 and 64.6; 20 x (2 + 10) x
//   1318, 256 (0.63, 18) 49.9 and 51.6; 4 x (3 + 13) x 4096, 128 (0.46, 16) 49.2 and 49.1; but 8 x (2 + 10) x 2048, 128 (0.39, 11)
//   35.0 and 31.5; 2 x (1 + 15) x 13337, 47 (0.1, 27) 73.5 and 65.6.
// * over all keys: the same from ten chunks on (10 x (2 + 10) x 1056, 256 (0.60, 9) 26.0 and 28.0; 3 x (2 + 10) x 8811, 256
//   (0.58, 18) 47.6 and 53.3; 6 x (2 + 10) x 2863, 64 (0.29, 12) 35.1 and 33.9), and of more pieces than units all of five chunks
//   on (32 x (3 + 9) x 577, 64 38.2 and 35.6; 31 x (1 + 15) x 695, 256 46.7 and 42.5; 45 x (1 + 15) x 437, 128, two to three pieces
//   a unit, 41.7 and 47.5).  Eight also beside more query blocks than that launch holds, where they weigh more than the chunks: 11 x
//   (11 + 5) x 8014, 282 256 and 223, 6 x (20 + 12) x 6407, 369 220 and 199, 21 x (12 + 4) x 595, 265 50.2 and 46.6; 13 x (13 + 3) x 644,
//   256 (pieces of two chunks) 36.3 and 36.4.
struct ReadOutCut {
  bool causal, mapped;   // mapped: features mapped beforehand
  long pieces, chunks;   // chunks of a piece
  long head;             // chunks of a head
  long sums;             // carried sums a piece starts from, at most
  long sum_blocks;       // sums of the state pass
  long sum_chunks;       // chunks of a sum
  long query_blocks;     // of the windowed heads, where they can share a launch
  long tiles;            // key tiles of a query block, at most
};
bool halves_apart(const ReadOutCut& c, long cus) {
  if (c.chunks == 1 || (c.causal ? c.chunks <= 4 && c.sums > c.chunks : 2 * c.sums > c.chunks)) return false;
  if (c.causal ? c.pieces > cus : c.mapped || (c.pieces > 2 * cus && c.pieces <= 3 * cus)) return false;
  if (c.query_blocks == 0) return true;
  if (c.sums == 0) return false;
  const long beside = c.query_blocks * c.tiles, own = c.pieces * c.chunks;
  const bool few = 5 * beside <= 2 * own, fits = c.pieces + c.query_blocks <= 2 * cus;
  if (!c.causal)
    return (c.pieces > cus ? c.chunks >= 5 : c.chunks >= 10 && few) || (c.chunks >= 4 && c.query_blocks > 3 * cus && beside >= own);
  if (2 * c.tiles > 3 * c.sum_chunks || (c.tiles > c.sum_chunks && 8 * c.sum_blocks < 5 * cus && fits)) return false;
  if (c.chunks > c.head && c.tiles < c.sum_chunks && beside >= own && 10 * (c.pieces + c.query_blocks) >= 19 * cus) return false;
  if (c.sum_chunks <= 4 && c.sum_blocks + c.query_blocks > 3 * cus && c.pieces + c.query_blocks <= 4 * cus &&
      (beside > 5 * own || 2 * c.sum_blocks > 3 * c.pieces))
    return false;
  if (c.mapped) return c.chunks >= 8 && few;
  return c.chunks >= 5 || (c.chunks == 4 && !fits);
}

// Shared by gformer_attn_plan, gformer_attn_workspace_bytes and gformer_attn_fwd.
// Token i of a windowed head sees keys i - left .. i + right (cut at the sequence ends): the w
// tokens ending at i, or (bidirectional) the w tokens centred on it.
// Both reaches are cut at N - 1 here, once: a token cannot see further than the sequence, and
// the tile arithmetic of the kernels and planners (reach + tile size, row + reach) then stays far
// from the end of the int range for any window up to INT_MAX (the natural way to ask for full
// attention).
int window_left(int window, int bidirectional, int N) {
  const int reach = bidirectional ? window / 2 : window - 1;
  return reach < N - 1 ? reach : (N > 1 ? N - 1 : 0);
}
int window_right(int window, int bidirectional, int N) {
  const int reach = bidirectional ? window - 1 - window / 2 : 0;
  return reach < N - 1 ? reach : (N > 1 ? N - 1 : 0);
}

// With short_pieces = false small calls are cut as they were before that rule existed: what a workspace
// sized for that cut still gets.
gf_status resolve(int B, int H, int N, int d, int window, const gformer_params* p, Resolved* r,
                  bool short_pieces = true) {
  memset(r, 0, sizeof(*r));
  if (!p) return GF_ERR_INVALID_ARG;
  if (p->struct_size != sizeof(gformer_params)) return GF_ERR_INVALID_ARG;
  if (B < 0 || H < 0 || N < 0 || d < 1 || window < 1) return GF_ERR_INVALID_ARG;
  if (p->dtype != GF_F32 && p->dtype != GF_BF16) return GF_ERR_INVALID_ARG;
  if (p->phi != GF_PHI_ELU1 && p->phi != GF_PHI_IDENTITY) return GF_ERR_INVALID_ARG;
  if (p->impl != GF_IMPL_AUTO && p->impl != GF_IMPL_SCALAR && p->impl != GF_IMPL_MFMA &&
      p->impl != GF_IMPL_MFMA_BLOCKED && p->impl != GF_IMPL_MFMA_STREAM &&
      p->impl != GF_IMPL_MFMA_CHUNK)
    return GF_ERR_INVALID_ARG;
  if (p->n_sparse_heads < 0 || p->n_sparse_heads > H) return GF_ERR_INVALID_ARG;
  if (p->chunk < 0 || p->segment_len < 0) return GF_ERR_INVALID_ARG;
  if (p->launch_mask < 0 || p->launch_mask > 7) return GF_ERR_INVALID_ARG;
  if (p->overlap != 0 && p->overlap != 1) return GF_ERR_INVALID_ARG;
  if (p->bidirectional != 0 && p->bidirectional != 1) return GF_ERR_INVALID_ARG;
  if (!(p->softmax_scale == p->softmax_scale) || !(p->eps >= 0.f)) return GF_ERR_INVALID_ARG;
  if (B > 65535 || H > 65535) return GF_ERR_UNSUPPORTED;  // grid y/z limits
  gf_status st;
  if ((st = check_strides(p->q_stride, r->qs, H, N, d)) != GF_OK) return st;
  if ((st = check_strides(p->k_stride, r->ks, H, N, d)) != GF_OK) return st;
  if ((st = check_strides(p->v_stride, r->vs, H, N, d)) != GF_OK) return st;
  if ((st = check_strides(p->o_stride, r->os, H, N, d)) != GF_OK) return st;
  if (d != 64 && d != 128) return GF_ERR_UNSUPPORTED;

  int impl = p->impl;
  if (impl == GF_IMPL_AUTO) impl = (p->dtype == GF_BF16) ? GF_IMPL_MFMA : GF_IMPL_SCALAR;
  // the others differ from GF_IMPL_MFMA only in which kernel runs the windowed heads or the
  // linear read-out
  if (impl == GF_IMPL_MFMA_BLOCKED || impl == GF_IMPL_MFMA_STREAM || impl == GF_IMPL_MFMA_CHUNK)
    impl = GF_IMPL_MFMA;
  if (impl == GF_IMPL_MFMA && p->dtype != GF_BF16) return GF_ERR_UNSUPPORTED;
  if (p->chunk != 0 && p->chunk != 64 && p->chunk != 128 && p->chunk != 256) return GF_ERR_UNSUPPORTED;

  gformer_plan& pl = r->plan;
  pl.impl = impl;
  const long kComputeUnits = device_compute_units();
  const int H0 = p->n_sparse_heads, H1 = H - H0;
  const long heads_lin = (long)B * H1;
  if (impl == GF_IMPL_SCALAR) {
    pl.chunk = 32;  // fixed by the fp32 kernels
    pl.segment_len = N;
    pl.n_segments = (H1 > 0 && N > 0) ? (int)heads_lin : 0;  // one workgroup walks a whole head
    if (p->segment_len != 0 && p->segment_len < N) return GF_ERR_UNSUPPORTED;
    pl.windowed_threads = kScalarThreads;
    pl.windowed_blocks = (H0 > 0 && N > 0) ? B * H0 * ((N + kScalarWindowRows - 1) / kScalarWindowRows) : 0;
    pl.linear_threads = kScalarThreads;
    pl.linear_blocks = (H1 > 0 && N > 0) ? (int)heads_lin : 0;
    pl.state_blocks = 0;
    pl.workspace_bytes = 0;
    r->f32 = f32_matrix(p, B, H, N);
    if (r->f32 && N > 0) {
      if (H0 > 0) {
        const int rows = f32_window_rows((int64_t)B * H0, N);
        pl.windowed_blocks = B * H0 * ((N + rows - 1) / rows);
      }
      if (H1 > 0) {
        const Segments f = f32_segments(heads_lin, N, d, p->bidirectional == 0, UINT64_MAX, 1);
        r->f32_seg_len = f.len;
        r->f32_nseg = f.count;
        pl.segment_len = f.len;
        pl.n_segments = pl.linear_blocks = (int)(heads_lin * f.count);
        pl.linear_threads = 4 * d;
        pl.state_blocks = (int)(heads_lin * (p->bidirectional ? f.count : f.count - 1));
        if (pl.state_blocks > 0)
          pl.workspace_bytes = r->needed = (uint64_t)pl.n_segments * ((uint64_t)d * d + d) * sizeof(float);
      }
    }
    return GF_OK;
  }
  pl.chunk = p->chunk ? p->chunk : 64;
  // Everything below counts in strips of 64 tokens (the tile every kernel works in); a chunk is
  // one, two or four of them.  Chunks of more than one strip (and GF_IMPL_MFMA_CHUNK at any
  // size) take the causal read-out to the general-chunk kernel, whose pieces are whole chunks of
  // one head.  The bidirectional read-out has no in-chunk part: there the chunk only sets the
  // granularity of segment_len.
  constexpr long kStrip = 64;
  const long cm = pl.chunk / kStrip;
  r->general_chunk = !p->bidirectional && (cm > 1 || p->impl == GF_IMPL_MFMA_CHUNK);
  if (r->general_chunk && H1 > 0 && !linear_chunk_supported(d, pl.chunk)) return GF_ERR_UNSUPPORTED;
  const long cph = N > 0 ? (N + kStrip - 1) / kStrip : 0;  // real strips per head
  pl.windowed_threads = kMfmaWindowThreads;
  const long query_blocks = (H0 > 0 && N > 0) ? (long)B * H0 * ((N + kMfmaWindowRows - 1) / kMfmaWindowRows) : 0;
  pl.windowed_blocks = (int)query_blocks;
  {
    const StreamPlan sp = windowed_stream_plan((int64_t)B * H0, N, window_left(window, p->bidirectional, N),
                                               window_right(window, p->bidirectional, N));
    if (p->impl == GF_IMPL_MFMA_STREAM && H0 > 0 && !sp.applies) return GF_ERR_UNSUPPORTED;
    r->stream = p->impl == GF_IMPL_MFMA_STREAM || (p->impl != GF_IMPL_MFMA_BLOCKED && sp.preferred);
    if (r->stream && H0 > 0 && N > 0) {
      pl.windowed_threads = sp.threads;
      pl.windowed_blocks = (int)sp.blocks;
    }
  }
  long piece = 0, vcph = cph, pieces = 0, mid = 0, sub = 1, most_sub = 0, carried = 0;
  // sums of equal pieces with no regard to heads, cut into n
  auto straddling_sums = [&](long n) {
    const long total = heads_lin * cph, ls = piece / n;
    long count = 0;
    for (long j = 1; j < pieces * n; ++j) {
      const long e = j * ls, next_main = (j + n - 1) / n * piece;
      count += (e % cph) != 0 && next_main < (e / cph + 1) * cph && next_main < total;
    }
    return count;
  };
  // sub-pieces of the `carried` pieces that the state pass sums, beside `blocks` others where the chip holds `room` of both
  auto cut_beside = [&](long blocks, long room) {
    long n = 4;
    while (n > 1 && !(piece % n == 0 && piece / n >= 4 && carried * n + blocks <= room)) n /= 2;
    return n;
  };
  if (p->segment_len != 0 && p->segment_len % pl.chunk != 0) return GF_ERR_INVALID_ARG;
  long own_piece = aligned_piece(heads_lin, cph, kComputeUnits);
  if (own_piece == 0 && !r->general_chunk && short_pieces) own_piece = short_piece(heads_lin, cph, kComputeUnits, d);
  if (p->bidirectional && heads_lin > 0 && cph > 0) {
    // Bidirectional linear heads: every piece needs the state of its whole head, so pieces never
    // straddle heads (uniform segments per head) and every one of them is summed by the state
    // pass.  Without a request: as many pieces per head as keep every compute unit at one piece.
    if (p->segment_len != 0) {
      piece = p->segment_len / kStrip;
    } else {
      long per = kComputeUnits / heads_lin;
      if (per < 1) per = 1;
      if (per > cph) per = cph;
      piece = (cph + per - 1) / per;
    }
    const long per_head = (cph + piece - 1) / piece;
    vcph = per_head * piece;
    pieces = heads_lin * per_head;
    mid = pieces;
  } else if (p->segment_len != 0 || (heads_lin > 0 && cph > 0 && (r->general_chunk || own_piece > 0))) {
    // Uniform segments per head: asked for, needed by the general-chunk kernel, or chosen
    // because a whole number of them per head keeps at least 4 of 5 compute units busy.  Pieces
    // that never straddle heads leave the state pass the least to re-read (a head's last segment
    // is never summed).
    piece = p->segment_len != 0 ? p->segment_len / kStrip : own_piece;
    if (piece == 0) {
      // general-chunk kernel with too few or too many heads for a good whole-number cut: as many
      // pieces per head as there are compute units for, none shorter than 8 strips
      long k = kComputeUnits / heads_lin;
      if (k > cph / 8) k = cph / 8;
      if (k < 1) k = 1;
      piece = (cph + k - 1) / k;
    }
    if (r->general_chunk) piece = (piece + cm - 1) / cm * cm;   // whole chunks
    const long per_head = cph > 0 ? (cph + piece - 1) / piece : 0;
    vcph = per_head * piece;
    pieces = heads_lin * per_head;
    // The state pass walks a head's segments but the last one.  A workgroup of it is bound by
    // its own chunk-by-chunk walk, so segments are cut into up to four sub-pieces as long as the
    // sub-pieces stay 4 chunks or longer and fit two workgroups per compute unit.
    carried = heads_lin * (per_head > 0 ? per_head - 1 : 0);
    sub = most_sub = cut_beside(0, 2 * kComputeUnits);
    mid = carried * sub;
  } else if (heads_lin > 0 && cph > 0) {
    // One workgroup per compute unit (its LDS holds one), each with the same number of chunks;
    // pieces no shorter than 8 chunks so the carried state (d*d fp32 in, d*d out) stays a small
    // share of the traffic.
    const long total = heads_lin * cph;
    piece = (total + kComputeUnits - 1) / kComputeUnits;
    if (piece < 8) piece = 8;
    if (piece > total) piece = total;
    if (piece % 2 != 0 && piece < total) ++piece;  // even, so the state pass can halve it
    pieces = (total + piece - 1) / piece;
    // Here the state pass works on half pieces (two workgroups per compute unit fit there), which
    // evens out its load: a sub-piece is summed iff a piece boundary follows it inside its head.
    sub = most_sub = piece % 2 == 0 ? 2 : 1;
    mid = straddling_sums(sub);
  }
  if (pieces > 0x7fffffffL / 64) return GF_ERR_UNSUPPORTED;
  r->cph = (int)cph;
  r->vcph = (int)vcph;
  r->piece_chunks = (int)piece;
  pl.segment_len = (int)(piece * kStrip);
  pl.n_segments = (int)pieces;
  // Where the query blocks share the state pass's launch and both fit the chip at once without a cut, the cut leaves room for
  // them.  d = 128, two on a unit: prefill of 2 x 32 x 3001, 156 sums of 12 chunks beside 288 query blocks 36 us, 312 of 6,
  // which need a second round, 43.  d = 64, three on a unit: uncut sums are few and long, so only where they come to three
  // of four units or have no more than 20 chunks.  The layer, us, finest cut and this: 1 x (2 + 10) x 18682 (240 sums of 12)
  // 52.0 and 44.6, 2 x (3 + 13) x 9000 (208 of 16) 63.3 and 58.7, 3 x (6 + 26) x 3750 (156 of 20) 69.3 and 63.3, 4 x (1 + 7) x 15727
  // (224 of 28) 79.5 and 80.1, but 8 x (2 + 10) x 4096 (160 of 22) 63.4 and 69.0, 11 x (1 + 7) x 5282 (154 of 28) 69.2 and 73.2.
  // Pieces across heads where they have no more than 20 chunks: 3 x (7 + 9) x 3096
  // (8 chunks) 1.25 times as fast, 5 x (3 + 13) x 3936 (16) 1.13, 9 x (2 + 10) x 3267 (20) 1.03, but 13 x (2 + 10) x 2520 (22) 0.99,
  // 19 x (1 + 7) x 2968 (26) 0.98, 9 x (1 + 31) x 6795 (118) 0.93.
  // The same cut where the query blocks have a launch of their own (negative scale, overlap, long sums): calls with a
  // launch mask, which share the sums, must agree on it, and it is no slower (finer, this: the same prefill's forward
  // with a negative scale 86.5, 78.5, with overlap 92.5, 81; 1 x 32 x 5338, H0 = 5 83.6, 76.1 and 85.3, 75.9; d = 64, apart
  // 1 x (2 + 10) x 18682 55.1, 53.7, 4 x (1 + 7) x 15727 83.5, 86.5).
  // The workspace reported has room for the sums of the finer cut, so that its size depends on the shape alone.
  const long room = (d == 128 ? 2 : 3) * kComputeUnits;
  long sub_beside = sub, mid_beside = mid;
  if (sub > 1 && query_blocks > 0 && !r->stream && !p->bidirectional) {
    if (carried > 0 && (d == 128 || 4 * carried >= 3 * kComputeUnits || piece <= 20)) {
      if (carried + query_blocks <= room) sub_beside = std::min(sub, cut_beside(query_blocks, room));
      mid_beside = carried * sub_beside;
    } else if (d == 64 && carried == 0 && piece <= 20 && mid + query_blocks > room) {
      const long whole = straddling_sums(1);
      if (whole + query_blocks <= room) {
        sub_beside = 1;
        mid_beside = whole;
      }
    }
  }
  r->query_halves = 1;
  if (d == 64 && pieces > 0) {
    long sums = mid > 0 ? sums_to_add(!p->bidirectional, (int)vcph, (int)piece, (int)(piece / sub)) : 0;
    if (mid > 0 && (sums == 0 || sums > sums_in_place(d))) sums = 1;   // scanned beforehand, where there are many
    const long reach = (long)window_left(window, p->bidirectional, N) + window_right(window, p->bidirectional, N);
    const long tiles = std::min((reach + kMfmaWindowRows - 1) / kStrip, (N - 1) / kStrip) + 1;
    const ReadOutCut c{!p->bidirectional, p->phi != GF_PHI_ELU1, pieces, piece, cph, sums, mid_beside, piece / sub_beside,
                       r->stream ? 0 : query_blocks, tiles};
    if (halves_apart(c, kComputeUnits)) r->query_halves = 2;
  }
  if (d == 128 || r->query_halves == 2) {
    sub = sub_beside;
    mid = mid_beside;
  }
  r->state_sub = (int)sub;
  pl.linear_threads = mfma_linear_threads(d, r->general_chunk ? 1 : r->query_halves);
  pl.linear_blocks = (int)pieces;
  pl.state_blocks = (int)mid;
  const uint64_t slots = mid > 0 ? (uint64_t)pieces * ((uint64_t)d * d + d) * sizeof(float) : 0;
  r->needed = slots * sub;
  pl.workspace_bytes = slots * (most_sub > 0 ? most_sub : sub);
  return GF_OK;
}

}  // namespace
}  // namespace gformer

using namespace gformer;

extern "C" {

void gformer_params_init(gformer_params* p) {
  if (!p) return;
  memset(p, 0, sizeof(*p));
  p->struct_size = sizeof(gformer_params);
  p->dtype = GF_BF16;
  p->phi = GF_PHI_ELU1;
  p->impl = GF_IMPL_AUTO;
  p->softmax_scale = 1.0f;
  p->eps = 0.0f;
}

size_t gformer_attn_workspace_bytes(int B, int H, int N, int d, int window,
                                    const gformer_params* p) {
  Resolved r;
  if (resolve(B, H, N, d, window, p, &r) != GF_OK) return 0;
  return (size_t)r.plan.workspace_bytes;
}

gf_status gformer_attn_plan(int B, int H, int N, int d, int window, const gformer_params* p,
                            gformer_plan* plan) {
  if (!plan) return GF_ERR_INVALID_ARG;
  Resolved r;
  gf_status st = resolve(B, H, N, d, window, p, &r);
  *plan = r.plan;
  return st;
}

}  // extern "C"

namespace {

// The whole layer; with rings / final states it also leaves what a decode step continues from.
gf_status attn_forward(const void* q, const void* k, const void* v, void* out, void* kring,
                       void* vring, float* final_state, int B, int H, int N, int d, int window,
                       const gformer_params* p, void* workspace, size_t workspace_bytes,
                       void* hip_stream) {
  Resolved r;
  gf_status st = resolve(B, H, N, d, window, p, &r);
  if (st != GF_OK) return st;
  // a workspace the short pieces cannot use (too small, or not aligned) still serves the longer cut, which often
  // needs none
  if (!r.f32 && r.needed > 0 && (!workspace || ((uintptr_t)workspace & 255u) || workspace_bytes < r.needed))
    st = resolve(B, H, N, d, window, p, &r, false);
  if (st != GF_OK) return st;
  if (B == 0 || H == 0 || N == 0) return GF_OK;
  if (!q || !k || !v || !out) return GF_ERR_INVALID_ARG;
  if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)out) & 15u) return GF_ERR_INVALID_ARG;
  if (out == q || out == k || out == v) return GF_ERR_INVALID_ARG;
  if (r.f32) {
    // The workspace is what lets a head be cut into segments; without one (or with a smaller one)
    // the layer is computed all the same, from fewer segments.
    if ((uintptr_t)workspace & 255u) workspace = nullptr;
    if (!workspace) workspace_bytes = 0;
    if (workspace_bytes < r.needed) {
      const int64_t heads = (int64_t)B * (H - p->n_sparse_heads);
      const Segments f = f32_segments(heads, N, d, p->bidirectional == 0, workspace_bytes, 1);
      r.f32_seg_len = f.len;
      r.f32_nseg = f.count;
    }
  } else if (r.needed > 0) {
    if (!workspace || workspace_bytes < r.needed) return GF_ERR_WORKSPACE;
    if ((uintptr_t)workspace & 255u) return GF_ERR_INVALID_ARG;
  }
  // only the kernel specialised for chunks of 64 writes the states a decode step continues from
  if (final_state && r.general_chunk && p->n_sparse_heads < H) return GF_ERR_UNSUPPORTED;

  AttnArgs a;
  memset(&a, 0, sizeof(a));
  a.q = TensorView{q, r.qs[0], r.qs[1], r.qs[2]};
  a.k = TensorView{k, r.ks[0], r.ks[1], r.ks[2]};
  a.v = TensorView{v, r.vs[0], r.vs[1], r.vs[2]};
  a.out = out;
  a.osb = r.os[0]; a.osh = r.os[1]; a.osn = r.os[2];
  a.B = B; a.H = H; a.N = N; a.d = d;
  a.window = window;
  a.causal = p->bidirectional ? 0 : 1;
  a.wleft = window_left(window, p->bidirectional, N);
  a.wright = window_right(window, p->bidirectional, N);
  a.H0 = p->n_sparse_heads;
  a.phi = p->phi;
  a.scale = p->softmax_scale;
  a.eps = p->eps;
  a.chunk = r.plan.chunk;
  a.cph = r.cph;
  a.vcph = r.vcph;
  a.piece_chunks = r.piece_chunks;
  a.n_pieces = r.plan.n_segments;
  a.state_sub = (int16_t)r.state_sub;
  a.query_halves = (int16_t)r.query_halves;
  a.f32_seg_len = r.f32_seg_len;
  a.f32_nseg = r.f32_nseg;
  a.ws_states = r.needed > 0 ? reinterpret_cast<float*>(workspace) : nullptr;
  a.final_state = final_state;
  a.kring = kring;
  a.vring = vring;

  hipStream_t s = reinterpret_cast<hipStream_t>(hip_stream);
  const int mask = p->launch_mask ? p->launch_mask : 7;
  const bool bf16 = p->dtype == GF_BF16;
  hipError_t e = hipSuccess;
  if (r.f32) {
    // the sums over all keys need a slot per head: the plain-FMA kernel keeps its own
    const uint64_t one = (uint64_t)B * (H - a.H0) * ((uint64_t)d * d + d) * sizeof(float);
    const bool plain = !a.causal && workspace_bytes < one;
    const bool together = (mask & GF_LAUNCH_WINDOWED) && (mask & GF_LAUNCH_LINEAR_MAIN) && !plain && !p->overlap &&
                          f32_takes_windowed(d, B, H, a.H0, N);
    if ((mask & GF_LAUNCH_WINDOWED) && !together) e = launch_windowed_f32(a, s);
    if ((mask & GF_LAUNCH_LINEAR_MAIN) && e == hipSuccess)
      e = plain ? launch_linear_scalar(a, bf16, s) : launch_linear_f32(a, together, s);
  } else if (r.plan.impl == GF_IMPL_SCALAR) {
    if ((mask & GF_LAUNCH_WINDOWED) && e == hipSuccess) e = launch_windowed_scalar(a, bf16, s);
    if ((mask & GF_LAUNCH_LINEAR_MAIN) && e == hipSuccess) e = launch_linear_scalar(a, bf16, s);
  } else {
    const bool win = (mask & GF_LAUNCH_WINDOWED) && a.H0 > 0;
    // large problems with windows of at most five key tiles stream; the rest goes query block
    // by query block
    const bool stream = r.stream;
    auto launch_windowed = [&](hipStream_t on) {
      return stream ? launch_windowed_stream(a, on) : launch_windowed_mfma(a, on);
    };
    const bool lin = (mask & (GF_LAUNCH_LINEAR_STATE | GF_LAUNCH_LINEAR_MAIN)) && a.H0 < a.H;
    std::lock_guard<std::mutex> lock(g_enqueue_mutex);
    SideStream* side = nullptr;
    if (win && lin && p->overlap) e = side_stream_for_current_device(s, &side);
    // The windowed heads' query blocks ride in the state pass's launch, but for long sums beside few blocks, or, beside a
    // four-wave read-out at d = 64, in that one's (halves_apart, linear_mfma.hip).  Not the
    // streaming kernel (other block size), a forced overlap, or a launch mask that names one of the two.
    const bool joint = win && !p->overlap && !stream;
    const bool together = joint && (mask & GF_LAUNCH_LINEAR_MAIN) && !r.general_chunk && linear_main_takes_windowed(a);
    const bool with_state = joint && (mask & GF_LAUNCH_LINEAR_STATE) && linear_state_takes_windowed(a);
    bool forked = false;
    if (side && e == hipSuccess) {
      // fork: the windowed heads wait for what is already in `s`, then run beside the linear ones
      e = hipEventRecord(side->fork, s);
      if (e == hipSuccess) e = hipStreamWaitEvent(side->stream, side->fork, 0);
      forked = e == hipSuccess;
      if (e == hipSuccess) e = launch_windowed(side->stream);
    }
    // The read-out kernel wants every compute unit at once (one piece each), so only the state
    // pass, whose small workgroups pack two to a unit, shares the chip with the windowed heads.
    if ((mask & GF_LAUNCH_LINEAR_STATE) && e == hipSuccess) e = launch_linear_state_mfma(a, with_state, s);
    if (forked) {
      // join, also after a failed launch: a side stream left waiting on the fork would break a
      // capture in progress and leave `s` unordered against what did get enqueued
      const hipError_t j1 = hipEventRecord(side->join, side->stream);
      const hipError_t j2 = j1 == hipSuccess ? hipStreamWaitEvent(s, side->join, 0) : j1;
      if (e == hipSuccess) e = j2;
    } else if (win && !side && !together && !with_state && e == hipSuccess) {
      e = launch_windowed(s);
    }
    if ((mask & GF_LAUNCH_LINEAR_MAIN) && e == hipSuccess)
      e = together ? launch_linear_main_windowed_mfma(a, s)
                   : r.general_chunk ? launch_linear_chunk(a, s) : launch_linear_main_mfma(a, s);
  }
  // (the query blocks of the bf16 kernels fill the rings themselves)
  if (e == hipSuccess && (r.plan.impl == GF_IMPL_SCALAR || r.stream)) e = launch_fill_rings(a, bf16, s);
  return e == hipSuccess ? GF_OK : GF_ERR_DEVICE;
}

}  // namespace

extern "C" {

gf_status gformer_attn_fwd(const void* q, const void* k, const void* v, void* out, int B, int H,
                           int N, int d, int window, const gformer_params* p, void* workspace,
                           size_t workspace_bytes, void* hip_stream) {
  return attn_forward(q, k, v, out, nullptr, nullptr, nullptr, B, H, N, d, window, p, workspace,
                      workspace_bytes, hip_stream);
}

gf_status gformer_attn_fwd_noalloc(const void* q, const void* k, const void* v, void* out, int B,
                                   int H, int N, int d, int window, const gformer_params* p,
                                   void* hip_stream) {
  Resolved r;
  const gf_status st = resolve(B, H, N, d, window, p, &r);
  if (st != GF_OK) return st;
  if (p->overlap != 0) return GF_ERR_UNSUPPORTED;   // the side stream is created on first use
  // (a single-precision call runs with whatever sums fit)
  if (!r.f32 && r.needed > kScratchBytes) return GF_ERR_WORKSPACE;
  if (B == 0 || H == 0 || N == 0) return GF_OK;
  void* ws = nullptr;
  if (r.needed > 0) {
    std::lock_guard<std::mutex> lock(g_enqueue_mutex);
    if (scratch_for_current_device(reinterpret_cast<hipStream_t>(hip_stream), &ws) != hipSuccess) {
      (void)hipGetLastError();
      return GF_ERR_DEVICE;
    }
  }
  return attn_forward(q, k, v, out, nullptr, nullptr, nullptr, B, H, N, d, window, p, ws,
                      ws ? kScratchBytes : 0, hip_stream);
}

gf_status gformer_attn_prefill(const void* q, const void* k, const void* v, void* out, void* kcache,
                               void* vcache, float* state, int B, int H, int N, int d, int window,
                               const gformer_params* p, void* workspace, size_t workspace_bytes,
                               void* hip_stream) {
  if (!p || p->struct_size != sizeof(gformer_params)) return GF_ERR_INVALID_ARG;
  if (p->bidirectional != 0 || p->launch_mask != 0) return GF_ERR_INVALID_ARG;
  if (B > 0 && H > 0 && N > 0) {
    const int H0 = p->n_sparse_heads;
    if (H0 > 0 && H0 <= H && (!kcache || !vcache)) return GF_ERR_INVALID_ARG;
    if (H0 >= 0 && H0 < H && !state) return GF_ERR_INVALID_ARG;
    if (((uintptr_t)kcache | (uintptr_t)vcache | (uintptr_t)state) & 15u) return GF_ERR_INVALID_ARG;
  }
  return attn_forward(q, k, v, out, kcache, vcache, state, B, H, N, d, window, p, workspace,
                      workspace_bytes, hip_stream);
}

gf_status gformer_attn_decode(const void* q, const void* k, const void* v, void* out, void* kcache,
                              void* vcache, float* state, int B, int H, int d, int window,
                              int64_t t, const gformer_params* p, void* hip_stream) {
  if (!p || p->struct_size != sizeof(gformer_params)) return GF_ERR_INVALID_ARG;
  if (B < 0 || H < 0 || d < 1 || window < 1 || t < 0) return GF_ERR_INVALID_ARG;
  if (p->dtype != GF_F32 && p->dtype != GF_BF16) return GF_ERR_INVALID_ARG;
  if (p->phi != GF_PHI_ELU1 && p->phi != GF_PHI_IDENTITY) return GF_ERR_INVALID_ARG;
  if (p->n_sparse_heads < 0 || p->n_sparse_heads > H) return GF_ERR_INVALID_ARG;
  if (!(p->softmax_scale == p->softmax_scale) || !(p->eps >= 0.f)) return GF_ERR_INVALID_ARG;
  if (p->bidirectional != 0) return GF_ERR_INVALID_ARG;   // a token cannot see what is not there yet
  if (B > 65535) return GF_ERR_UNSUPPORTED;
  if (d != 64 && d != 128) return GF_ERR_UNSUPPORTED;
  const int H0 = p->n_sparse_heads;
  if (decode_smem_bytes(d, window, H0) > 64 * 1024) return GF_ERR_UNSUPPORTED;  // ring scores in LDS
  if (B == 0 || H == 0) return GF_OK;
  if (!q || !k || !v || !out) return GF_ERR_INVALID_ARG;
  if (H0 > 0 && (!kcache || !vcache)) return GF_ERR_INVALID_ARG;
  if (H0 < H && !state) return GF_ERR_INVALID_ARG;
  if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)out | (uintptr_t)kcache |
       (uintptr_t)vcache | (uintptr_t)state) & 15u)
    return GF_ERR_INVALID_ARG;
  if (out == q || out == k || out == v) return GF_ERR_INVALID_ARG;

  DecodeArgs a;
  memset(&a, 0, sizeof(a));
  a.q = q; a.k = k; a.v = v; a.out = out;
  a.kcache = kcache; a.vcache = vcache; a.state = state;
  a.B = B; a.H = H; a.d = d; a.window = window; a.H0 = H0; a.phi = p->phi;
  a.t = t;
  a.scale = p->softmax_scale;
  a.eps = p->eps;
  const hipError_t e = launch_decode(a, p->dtype == GF_BF16, reinterpret_cast<hipStream_t>(hip_stream));
  return e == hipSuccess ? GF_OK : GF_ERR_DEVICE;
}

void gformer_feature_params_init(gformer_feature_params* p) {
  if (!p) return;
  memset(p, 0, sizeof(*p));
  p->struct_size = sizeof(gformer_feature_params);
  p->dtype = GF_BF16;
  p->impl = GF_IMPL_AUTO;
}

gf_status gformer_random_features(const void* x, const void* w, void* out, int B, int H, int N,
                                  int d, int m, const gformer_feature_params* p, void* hip_stream) {
  if (!p || p->struct_size != sizeof(gformer_feature_params)) return GF_ERR_INVALID_ARG;
  if (B < 0 || H < 0 || N < 0 || d < 1 || m < 1) return GF_ERR_INVALID_ARG;
  if (p->dtype != GF_F32 && p->dtype != GF_BF16) return GF_ERR_INVALID_ARG;
  if (p->impl != GF_IMPL_AUTO && p->impl != GF_IMPL_SCALAR && p->impl != GF_IMPL_MFMA)
    return GF_ERR_INVALID_ARG;
  if (p->head_begin < 0 || p->head_end < p->head_begin || p->head_end > H) return GF_ERR_INVALID_ARG;
  if (B > 65535 || H > 65535) return GF_ERR_UNSUPPORTED;
  int64_t xs[3], os[3];
  gf_status st;
  if ((st = check_strides(p->x_stride, xs, H, N, d)) != GF_OK) return st;
  if ((st = check_strides(p->o_stride, os, H, N, m)) != GF_OK) return st;
  if (m != d || (d != 64 && d != 128)) return GF_ERR_UNSUPPORTED;
  int impl = p->impl;
  if (impl == GF_IMPL_AUTO) impl = (p->dtype == GF_BF16) ? GF_IMPL_MFMA : GF_IMPL_SCALAR;
  if (impl == GF_IMPL_MFMA && p->dtype != GF_BF16) return GF_ERR_UNSUPPORTED;
  if (B == 0 || N == 0 || p->head_end == p->head_begin) return GF_OK;
  if (!x || !w || !out) return GF_ERR_INVALID_ARG;
  if (((uintptr_t)x | (uintptr_t)w | (uintptr_t)out) & 15u) return GF_ERR_INVALID_ARG;
  if (out == w) return GF_ERR_INVALID_ARG;
  // in place is fine only when every element keeps its address
  if (out == x && (xs[0] != os[0] || xs[1] != os[1] || xs[2] != os[2])) return GF_ERR_INVALID_ARG;
  if ((int64_t)B * (p->head_end - p->head_begin) * N > 0x7fffffffLL) return GF_ERR_UNSUPPORTED;

  FeatureArgs a;
  memset(&a, 0, sizeof(a));
  a.x = TensorView{x, xs[0], xs[1], xs[2]};
  a.w = w;
  a.out = out;
  a.osb = os[0]; a.osh = os[1]; a.osn = os[2];
  a.B = B; a.H = H; a.N = N; a.d = d;
  a.head_begin = p->head_begin;
  a.head_end = p->head_end;
  const hipError_t e = launch_random_features(a, p->dtype == GF_BF16, impl == GF_IMPL_MFMA,
                                              reinterpret_cast<hipStream_t>(hip_stream));
  return e == hipSuccess ? GF_OK : GF_ERR_DEVICE;
}

namespace {
// per-token statistics [B, H, N, 2] fp32, rounded up to 256 bytes
size_t bwd_stats_bytes(int B, int H, int N) {
  return ((size_t)B * H * N * 2 * sizeof(float) + 255) / 256 * 256;
}
// bf16: the carried sums of the segments
size_t bwd_segment_bytes(int64_t heads, const Segments& f, int d, bool causal) {
  if (causal && f.count == 1) return 0;
  return (size_t)heads * f.count * 2 * ((size_t)d * d + d) * sizeof(float);
}
// what a call cannot do without; a single-precision call cuts its heads into as many segments as the
// rest of the workspace holds sums for
size_t bwd_least_bytes(int B, int H, int N, int d, const gformer_params* p) {
  size_t need = bwd_stats_bytes(B, H, N);
  // bidirectional linear heads: the two d x d sums (and their vectors) of every head, each in up
  // to kBidirStateSlots per-segment partials
  if (p && p->bidirectional == 1 && p->n_sparse_heads >= 0 && p->n_sparse_heads < H && d > 0)
    need += (size_t)B * (H - p->n_sparse_heads) * 2 * kBidirStateSlots * ((size_t)d * d + d) * sizeof(float);
  return need;
}
}  // namespace

size_t gformer_attn_bwd_workspace_bytes(int B, int H, int N, int d, int window,
                                        const gformer_params* p) {
  (void)window;
  if (B <= 0 || H <= 0 || N <= 0) return 0;
  size_t need = bwd_stats_bytes(B, H, N);
  if (p && p->dtype == GF_F32 && p->impl == GF_IMPL_AUTO && p->n_sparse_heads >= 0 && p->n_sparse_heads < H && d > 0) {
    // single precision on the matrix cores: two carried sums per segment (what the call needs is less,
    // see gformer_attn_bwd)
    const int64_t heads = (int64_t)B * (H - p->n_sparse_heads);
    const Segments f = f32_segments(heads, N, d, p->bidirectional == 0, UINT64_MAX, 2);
    const size_t sums = (size_t)heads * f.count * 2 * ((size_t)d * d + d) * sizeof(float);
    const size_t least = bwd_least_bytes(B, H, N, d, p);
    if (f.count > 1 || p->bidirectional == 1) need += sums;
    return need > least ? need : least;
  }
  if (p && p->dtype == GF_BF16 && p->impl != GF_IMPL_SCALAR && d == 64 && p->n_sparse_heads >= 0 && p->n_sparse_heads < H) {
    // room for the most segments a call of this shape is cut into, with its windowed heads in launches of their own
    const int64_t heads = (int64_t)B * (H - p->n_sparse_heads);
    const bool causal = p->bidirectional == 0;
    const size_t sums = bwd_segment_bytes(heads, backward_segments(heads, N, d, causal, 0), d, causal);
    const size_t least = bwd_least_bytes(B, H, N, d, p);
    return need + sums > least ? need + sums : least;
  }
  return bwd_least_bytes(B, H, N, d, p);
}

gf_status gformer_attn_bwd(const void* q, const void* k, const void* v, const void* dout, void* dq,
                           void* dk, void* dv, int B, int H, int N, int d, int window,
                           const gformer_params* p, void* workspace, size_t workspace_bytes,
                           void* hip_stream) {
  if (!p) return GF_ERR_INVALID_ARG;
  if (p->struct_size != sizeof(gformer_params)) return GF_ERR_INVALID_ARG;
  // a call runs on the matrix-core kernels (bf16: AUTO, MFMA; fp32: AUTO) unless SCALAR asks for the
  // plain-FMA kernels
  if (p->impl == GF_IMPL_MFMA_BLOCKED || p->impl == GF_IMPL_MFMA_STREAM ||
      p->impl == GF_IMPL_MFMA_CHUNK)
    return GF_ERR_UNSUPPORTED;
  if (p->impl == GF_IMPL_MFMA && p->dtype != GF_BF16) return GF_ERR_UNSUPPORTED;
  gformer_params pp = *p;
  pp.impl = GF_IMPL_SCALAR;
  pp.segment_len = 0;
  Resolved r;
  const gf_status st = resolve(B, H, N, d, window, &pp, &r);
  if (st != GF_OK) return st;
  if (p->launch_mask != 0) return GF_ERR_INVALID_ARG;
  if (B == 0 || H == 0 || N == 0) return GF_OK;
  if (!q || !k || !v || !dout || !dq || !dk || !dv) return GF_ERR_INVALID_ARG;
  const void* ins[4] = {q, k, v, dout};
  void* outs[3] = {dq, dk, dv};
  for (const void* x : ins)
    if ((uintptr_t)x & 15u) return GF_ERR_INVALID_ARG;
  for (void* y : outs) {
    if ((uintptr_t)y & 15u) return GF_ERR_INVALID_ARG;
    for (const void* x : ins)
      if (x == y) return GF_ERR_INVALID_ARG;
  }
  if (dq == dk || dq == dv || dk == dv) return GF_ERR_INVALID_ARG;
  const size_t need = bwd_least_bytes(B, H, N, d, p);
  if (!workspace || workspace_bytes < need) return GF_ERR_WORKSPACE;
  if ((uintptr_t)workspace & 255u) return GF_ERR_INVALID_ARG;

  BwdArgs a;
  memset(&a, 0, sizeof(a));
  a.q = TensorView{q, r.qs[0], r.qs[1], r.qs[2]};
  a.k = TensorView{k, r.ks[0], r.ks[1], r.ks[2]};
  a.v = TensorView{v, r.vs[0], r.vs[1], r.vs[2]};
  a.dout = TensorView{dout, r.os[0], r.os[1], r.os[2]};
  a.dq = dq; a.dk = dk; a.dv = dv;
  a.B = B; a.H = H; a.N = N; a.d = d;
  a.window = window < N ? window : N;   // a wider window sees no more keys; keeps row + window in range
  a.causal = p->bidirectional ? 0 : 1;
  a.wleft = window_left(window, p->bidirectional, N);
  a.wright = window_right(window, p->bidirectional, N);
  a.H0 = p->n_sparse_heads;
  a.phi = p->phi;
  a.scale = p->softmax_scale;
  a.eps = p->eps;
  a.ws = reinterpret_cast<float*>(workspace);
  a.ws_state = a.causal ? nullptr
                        : reinterpret_cast<float*>(static_cast<char*>(workspace) + bwd_stats_bytes(B, H, N));
  const bool bf16 = p->dtype == GF_BF16;
  const bool mfma = bf16 && p->impl != GF_IMPL_SCALAR;
  // d = 64: the segment walks take the linear heads.  A causal call whose workspace does not hold their sums, or
  // with more heads than one grid dimension holds, gets the scans that sum what lies in front of (behind) a segment
  // again; over all keys the least workspace holds the sums, and so many heads would need 550 GB of it.
  const int64_t lin_heads = (int64_t)B * (H - a.H0);
  const bool one_grid = lin_heads < (1 << 22);
  if (mfma && d == 64 && !a.causal && !one_grid) return GF_ERR_UNSUPPORTED;
  const int64_t band_tiles = p->overlap || a.H0 <= 0 ? 0 : backward_band_tiles((int64_t)B * a.H0, N, a.wleft, a.wright);
  const Segments segs = backward_segments(lin_heads, N, d, a.causal, band_tiles);
  const bool segments = d == 64 && one_grid &&
                        workspace_bytes >= bwd_stats_bytes(B, H, N) + bwd_segment_bytes(lin_heads, segs, d, a.causal);
  // The linear heads' launches take the windowed heads' passes along: the walks all four, the d = 128 scans
  // three behind a launch for the statistics.
  const bool together = (segments || (d == 128 && a.causal && (int64_t)B * H < (1 << 20))) && a.H0 > 0 && a.H0 < a.H &&
                        !p->overlap && (int64_t)B * a.H0 * ((N + 127) / 128) < (1 << 21);
  auto launch_linear = [&](hipStream_t on) {
    if (segments) {
      a.ws_state = reinterpret_cast<float*>(static_cast<char*>(workspace) + bwd_stats_bytes(B, H, N));
      a.lin_segment_len = segs.len;
      a.lin_segments = segs.count;
      return launch_linear_backward_segments(a, together, on);
    }
    return a.causal ? launch_linear_backward_mfma(a, together, on) : launch_linear_backward_bidir_mfma(a, on);
  };
  hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);
  hipError_t e = hipSuccess;
  if (f32_matrix(p, B, H, N)) {
    a.ws_state = reinterpret_cast<float*>(static_cast<char*>(workspace) + bwd_stats_bytes(B, H, N));
    const Segments f = f32_segments(lin_heads, N, d, a.causal, workspace_bytes - bwd_stats_bytes(B, H, N), 2);
    a.f32_seg_len = f.len;
    a.f32_nseg = f.count;
    const bool f32_together = !p->overlap && f32_takes_windowed(d, B, H, a.H0, N);
    if (!f32_together) e = launch_windowed_backward_f32(a, stream);
    if (e == hipSuccess) e = launch_linear_backward_f32(a, f32_together, stream);
  } else if (mfma) {
    // The linear scans are one workgroup per head and segment: with fewer of those than compute
    // units the rest of the chip is idle for their whole duration.  With overlap = 1 the windowed
    // heads' passes therefore run beside them on the library's side stream (forked from and
    // joined to the caller's stream by events), and the scans are enqueued first so that their
    // workgroups get their compute units.  Without it the passes ride in the walks' and the scans'
    // launches (`together`) or are launches of their own in front of them.
    const bool both = a.H0 > 0 && a.H0 < a.H;
    std::lock_guard<std::mutex> lock(g_enqueue_mutex);
    SideStream* side = nullptr;
    if (both && p->overlap) e = side_stream_for_current_device(stream, &side);
    if (side && e == hipSuccess) {
      e = hipEventRecord(side->fork, stream);
      if (e == hipSuccess) {
        e = launch_linear(stream);
        hipError_t f = hipStreamWaitEvent(side->stream, side->fork, 0);
        if (f == hipSuccess) {
          if (e == hipSuccess) e = launch_windowed_backward_mfma(a, side->stream);
          // join whatever happened after the fork
          f = hipEventRecord(side->join, side->stream);
          if (f == hipSuccess) f = hipStreamWaitEvent(stream, side->join, 0);
        }
        if (e == hipSuccess) e = f;
      }
    } else if (e == hipSuccess) {
      if (!together || !segments) e = launch_windowed_backward_mfma(a, stream, together);
      if (e == hipSuccess) e = launch_linear(stream);
    }
  } else if (a.causal) {
    e = launch_backward_scalar(a, bf16, true, true, stream);
  } else {
    e = launch_backward_scalar(a, bf16, true, false, stream);   // the windowed heads
    if (e == hipSuccess) e = launch_linear_backward_bidir(a, bf16, stream);
  }
  return e == hipSuccess ? GF_OK : GF_ERR_DEVICE;
}

const char* gformer_status_string(gf_status s) {
  switch (s) {
    case GF_OK: return "ok";
    case GF_ERR_INVALID_ARG: return "invalid argument";
    case GF_ERR_UNSUPPORTED: return "unsupported configuration";
    case GF_ERR_WORKSPACE: return "workspace missing or too small";
    case GF_ERR_DEVICE: return "HIP launch or runtime failure";
  }
  return "unknown status";
}

int gformer_version(void) { return 100; }

}  // extern "C"
