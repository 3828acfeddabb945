// Shared host/device declarations of the GFormer attention library (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gformer {

// One [B,H,N,d] tensor: element (b,h,n,c) at base + b*sb + h*sh + n*sn + c (elements).
struct TensorView {
  const void* base;
  int64_t sb, sh, sn;
};

// Everything a kernel needs to know about one attention call.
struct AttnArgs {
  TensorView q, k, v;
  void* out;
  int64_t osb, osh, osn;
  int B, H, N, d;
  int window;
  int causal;        // 1: causal (window ends at the token, linear prefix); 0: bidirectional
  int wleft, wright; // windowed heads: token i sees keys i - wleft .. i + wright (cut at the ends)
  int H0;            // heads [0,H0) windowed, [H0,H) linear
  int phi;           // gf_phi
  float scale;       // softmax scale (windowed heads)
  float eps;         // linear denominator epsilon
  // Linear-attention work split.  The chunks (64 tokens) of all linear heads form one list in
  // which head i owns virtual chunks [i*vcph, (i+1)*vcph), the first `cph` of them real.  The
  // list is cut into `n_pieces` pieces of `piece_chunks` chunks; one workgroup walks one piece.
  // vcph == cph: pieces are cut with no regard to head boundaries (balanced);
  // vcph  > cph: every head is padded to a whole number of pieces (uniform segments per head).
  int chunk;         // tokens per chunk of the causal read-out (64, 128, 256)
  // the four counts below are in strips of 64 tokens whatever the chunk ("chunks" of the fixed-64 kernels)
  int cph;           // real strips per head = ceil(N / 64)
  int vcph;          // virtual chunks per head
  int piece_chunks;  // chunks per piece
  int n_pieces;      // pieces = workgroups of the read-out kernel
  int16_t state_sub;     // the state pass cuts every piece into this many equal sub-pieces (1, 2 or 4)
  int16_t query_halves;  // the read-out's matrix waves, in sets: 2 (d = 64) where they split a chunk's queries
  float* final_state; // optional [B*(H-H0), d*d + d] fp32: every linear head's (A, Z) after its last
                     // token, A row-major [feature][value] (what the decode step carries on from)
  void *kring, *vring; // optional [B, H0, window, d] rings: the last `window` keys / values of every
                     // windowed head, token t in slot t % window
  // Streaming windowed kernel: every (batch, windowed head) is cut into `win_pieces_per_head`
  // pieces of `win_pairs_per_piece` pairs of 32-query groups (set by its launcher).
  int win_pairs_per_piece, win_pieces_per_head;
  // Single-precision matrix-core kernels: every linear head in f32_nseg segments of f32_seg_len tokens
  // (a multiple of 32 unless there is one); ws_states holds [B*(H-H0)][f32_nseg][d*d + d] fp32 sums.
  int f32_seg_len, f32_nseg;
  float* ws_states;  // [n_pieces*state_sub, d*d + d] fp32: slot j = (A, Z) of its head just
                     // before global chunk j*piece_chunks/state_sub (piece p reads slot p*state_sub)
};
static_assert(sizeof(AttnArgs) <= 248, "with two ints beside it a launch's arguments are four cache lines");

// Sub-piece sums of `ls` chunks that a piece of `piece` chunks starts from, at most (0 for one where heads are no longer than `ls`).
__host__ __device__ inline int sums_to_add(bool causal, int vcph, int piece, int ls) {
  if (!causal) return vcph / ls;   // every piece adds up its whole head
  // a causal piece adds up the sub-pieces in front of it inside its head; the latest start is
  // the head's last piece when pieces never straddle heads, else the head's last chunk
  return (vcph % piece == 0 ? vcph - piece : vcph - 1) / ls;
}
// With few carried boundaries per head the read-out kernel adds up the per-sub-piece sums
// itself (independent loads, no extra launch); with many, a prefix kernel runs first and the
// read-out kernel reads a single slot.
__host__ __device__ inline int sums_in_place(int d) { return d == 64 ? 8 : 6; }   // sums of 16 KB and of 66 KB
__host__ __device__ inline bool uses_prefix_kernel(const AttnArgs& a) {
  return sums_to_add(a.causal, a.vcph, a.piece_chunks, a.piece_chunks / a.state_sub) > sums_in_place(a.d);
}

// bf16 storage helpers (round to nearest even on store).
__device__ __forceinline__ float bf16_bits_to_float(uint16_t b) {
  return __uint_as_float(((uint32_t)b) << 16);
}
__device__ __forceinline__ uint16_t float_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);  // quiet NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

template <typename T> struct Storage;
template <> struct Storage<float> {
  static __device__ __forceinline__ float load(const void* p, int64_t i) {
    return reinterpret_cast<const float*>(p)[i];
  }
  static __device__ __forceinline__ void store(void* p, int64_t i, float v) {
    reinterpret_cast<float*>(p)[i] = v;
  }
};
template <> struct Storage<uint16_t> {  // bf16 bit patterns
  static __device__ __forceinline__ float load(const void* p, int64_t i) {
    return bf16_bits_to_float(reinterpret_cast<const uint16_t*>(p)[i]);
  }
  static __device__ __forceinline__ void store(void* p, int64_t i, float v) {
    reinterpret_cast<uint16_t*>(p)[i] = float_to_bf16_bits(v);
  }
};

// One call of the backward pass: q, k, v and the gradient dout of the output in; dq, dk, dv out
// (dq is laid out like q, dk like k, dv like v).
struct BwdArgs {
  TensorView q, k, v, dout;
  void *dq, *dk, *dv;
  int B, H, N, d;
  int window;         // causal calls: tokens in the window, cut at N
  int wleft, wright;  // windowed heads: token i sees keys i - wleft .. i + wright (cut at the ends)
  int causal;         // 1: causal layer; 0: bidirectional (centred window, linear heads over all keys)
  int H0;
  int phi;
  float scale, eps;
  float* ws_state;    // bidirectional linear heads (plain-FMA kernels, and the bf16 sweeps of d = 128):
                      // [B * (H - H0)][2][4][d*d + d] fp32: the sums
                      // (S, z) and (B, Y) of every head, each in up to four per-segment partials
                      // (matrix row-major [feature][value], then the vector)
  // single-precision matrix-core kernels: segments as in AttnArgs; ws_state holds the sums (A, Z) and
  // then (B, Y) of every segment, [2][B*(H-H0)][f32_nseg][d*d + d] fp32
  int f32_seg_len, f32_nseg;
  int lin_segment_len;  // bf16 segment walks: tokens per segment (a multiple of 32 unless there is one)
  int lin_segments;   // workgroups per linear head in the matrix-core scans (set by their launcher)
  int lin_bounds[5];  // segment s covers chunks [lin_bounds[s], lin_bounds[s+1]) (reverse scan: mirrored)
  float* ws;   // [B, H, N, 2] fp32: windowed heads (log-sum-exp, dO.o), linear heads (den, dO.o / den),
               // written by the per-query kernels, read by the per-key kernels
};
// plain-FMA kernels: the windowed heads, the linear heads, or both
hipError_t launch_backward_scalar(const BwdArgs& a, bool bf16, bool windowed_heads, bool linear_heads,
                                  hipStream_t s);
// bf16 matrix-core kernels for the windowed heads and for the linear heads
hipError_t launch_windowed_backward_mfma(const BwdArgs& a, hipStream_t s, bool statistics_only = false);
// with_windowed (d = 128): the windowed heads' dq, dk and dv passes ride in the scans' launches; their
// statistics have to be there.
hipError_t launch_linear_backward_mfma(const BwdArgs& a, bool with_windowed, hipStream_t s);
// bidirectional linear heads: plain-FMA kernels on either storage type, matrix-core kernels (bf16)
hipError_t launch_linear_backward_bidir(const BwdArgs& a, bool bf16, hipStream_t s);
hipError_t launch_linear_backward_bidir_mfma(const BwdArgs& a, hipStream_t s);
constexpr int kBidirStateSlots = 4;   // per-segment partials kept per sum

// One call of the random-feature pre-map: heads [head_begin, head_end) of x -> the same heads of out.
struct FeatureArgs {
  TensorView x;
  const void* w;     // [d, d] row-major, same element type as x
  void* out;
  int64_t osb, osh, osn;
  int B, H, N, d;
  int head_begin, head_end;
};

// One decode step: the new token of every (batch, head), the windowed heads' key/value rings
// and the linear heads' carried states.
struct DecodeArgs {
  const void *q, *k, *v;   // [B, H, d] dense
  void* out;               // [B, H, d] dense
  void *kcache, *vcache;   // [B, H0, window, d] dense rings
  float* state;            // [B, H - H0, d*d + d] fp32: A row-major [feature][value], then Z
  int B, H, d, window, H0, phi;
  int64_t t;               // position of the token, 0-based
  float scale, eps;
};

// Host-side launchers, one per kernel family.  Each returns the hipError_t of its launch.
hipError_t launch_windowed_scalar(const AttnArgs& a, bool bf16, hipStream_t s);
hipError_t launch_linear_scalar(const AttnArgs& a, bool bf16, hipStream_t s);
hipError_t launch_windowed_mfma(const AttnArgs& a, hipStream_t s);
// The streaming form of the same heads, for windows that span at most kStreamSlots key tiles.
constexpr int kStreamSlots = 5;
struct StreamPlan {
  bool applies;          // the window fits the kernel
  bool preferred;        // ... and the problem is large enough for it to beat the query-block kernel
  int pairs_per_piece;   // 64-query pairs one workgroup walks
  int pieces_per_head;
  int64_t blocks;        // workgroups = heads * pieces_per_head
  int threads;
};
StreamPlan windowed_stream_plan(int64_t heads, int N, int wleft, int wright);
hipError_t launch_windowed_stream(const AttnArgs& a, hipStream_t s);
// with_windowed: the windowed heads' query blocks ride in the state pass's launch, where that takes them along.
bool linear_state_takes_windowed(const AttnArgs& a);
hipError_t launch_linear_state_mfma(const AttnArgs& a, bool with_windowed, hipStream_t s);
hipError_t launch_linear_main_mfma(const AttnArgs& a, hipStream_t s);
// The read-out and the windowed heads' query blocks in one launch, where the former takes them along.
bool linear_main_takes_windowed(const AttnArgs& a);
hipError_t launch_linear_main_windowed_mfma(const AttnArgs& a, hipStream_t s);
// The causal read-out for chunks of 64, 128 or 256 tokens (the general form of the kernel above).
bool linear_chunk_supported(int d, int chunk);
hipError_t launch_linear_chunk(const AttnArgs& a, hipStream_t s);
hipError_t launch_fill_rings(const AttnArgs& a, bool bf16, hipStream_t s);
hipError_t launch_random_features(const FeatureArgs& a, bool bf16, bool mfma, hipStream_t s);
hipError_t launch_decode(const DecodeArgs& a, bool bf16, hipStream_t s);
size_t decode_smem_bytes(int d, int window, int H0);

// Single-precision matrix-core kernels.  A head's segments: at most three workgroups on every
// compute unit, none shorter than 128 tokens, as far as `bytes` hold `sums` carried sums for each.
constexpr int kMaxSegments = 64;
struct Segments {
  int len, count;
};
Segments f32_segments(int64_t heads, int N, int d, bool causal, uint64_t bytes, int sums);
// In place over [heads][nseg][floats]: mode 0, the sum over the slots before each; 1, behind each; 2, slot 0
// receives the total.
hipError_t launch_segment_scan(float* sums, int heads, int nseg, int floats, int mode, hipStream_t s);
int f32_window_rows(int64_t heads, int N);   // resident rows per workgroup of the windowed kernels
hipError_t launch_windowed_f32(const AttnArgs& a, hipStream_t s);
// with_windowed: the windowed heads' workgroups ride in the walks' launches, where f32_takes_windowed allows it
bool f32_takes_windowed(int d, int B, int H, int H0, int N);
hipError_t launch_linear_f32(const AttnArgs& a, bool with_windowed, hipStream_t s);
hipError_t launch_windowed_backward_f32(const BwdArgs& a, hipStream_t s);
hipError_t launch_linear_backward_f32(const BwdArgs& a, bool with_windowed, hipStream_t s);
// bf16 backward pass of the linear heads at d = 64, heads cut into segments (lin_segments of lin_segment_len
// tokens); ws_state holds [2][B*(H-H0)][lin_segments][d*d + d] fp32 sums unless there is one causal segment.
// band_tiles: 64-row tiles that a pass over the windowed heads' band walks in the same launches (0: none ride along).
Segments backward_segments(int64_t heads, int N, int d, bool causal, int64_t band_tiles);
int64_t backward_band_tiles(int64_t windowed_heads, int N, int wleft, int wright);
// with_windowed: the windowed heads' passes ride in the same launches.
hipError_t launch_linear_backward_segments(const BwdArgs& a, bool with_windowed, hipStream_t s);
constexpr int64_t kF32MaxRows = (int64_t)1 << 26;   // B * heads * N / 16 workgroups stay inside a grid

// Dynamic LDS of a launch.  Up to 64 KB in all (a kernel's static arrays take a few bytes beside it) need not be asked
// for, which saves a call into the runtime per launch (a training step of
// 32 x 12 x 577 x 64, whose host side is what it takes: 143.4 -> 141.3 us).
template <typename K> hipError_t allow_lds(K kern, size_t bytes) {
  if (bytes <= 60 * 1024) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// Launch geometry shared by the planner and the launchers.
constexpr int kScalarWindowRows = 16;   // query rows per workgroup, scalar windowed kernel
constexpr int kScalarThreads = 256;
constexpr int kMfmaWindowRows = 128;    // query rows per workgroup, MFMA windowed kernel
constexpr int kMfmaWindowThreads = 256;
int mfma_linear_threads(int d, int query_halves);   // of a read-out's workgroup
int device_compute_units();   // of the current device; 256 (MI355X) in a process without one

}  // namespace gformer
