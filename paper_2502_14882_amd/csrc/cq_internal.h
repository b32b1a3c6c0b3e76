// Internal declarations shared by the host API and the HIP kernels of libcq.
// Not part of the ABI (see include/cq.h for that).
#ifndef CQ_INTERNAL_H_
#define CQ_INTERNAL_H_

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "cq.h"
#include "cq_bench.h"

namespace cq {

// Tokens per block-level work item of the decode pipeline.  A "chunk" is the unit of
// split-K: every chunk produces one (m, l, acc[d]) partial of the online softmax.
constexpr int kVisChunk = 512;
constexpr int kTextChunk = 512;
constexpr int kMaxTileChunks = 64;   // tile kernels: most chunks per row, of the visual tokens and of the tail

struct DecodeShape {
  // n_text: tokens of the fp16 tail that are attended, or - when the length lives in device
  // memory (n_text_dev below) - the host's upper bound of it, which sizes launches and buffers
  int B, Hq, Hkv, g, d, n_vis, n_text, n_text_cap;
  int bits, k_axis, v_axis, k_group, v_group;
  int n_vis_chunks, n_text_chunks, n_chunks;
  int words_per_token;  // d * bits / 32
};

// Layout of the caller-provided workspace (all float, offsets in floats).
struct Workspace {
  size_t logits;    // [B][Hq][n_vis + n_text]       raw (uncalibrated) logits
  size_t minmax;    // [B][Hq][n_chunks][2]          min, max of each chunk's logits
  size_t partial;   // [B][Hq][n_chunks][d + 2]      m, l, acc[d]
  size_t total_bytes;
};

inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

inline Workspace workspace_layout(int B, int Hq, int d, int n_vis, int n_text) {
  Workspace w;
  const int nvc = ceil_div(n_vis, kVisChunk), ntc = ceil_div(n_text, kTextChunk);
  const size_t rows = (size_t)B * (size_t)Hq;
  auto align64 = [](size_t x) { return (x + 63) / 64 * 64; };
  w.logits = 0;
  w.minmax = align64(w.logits + rows * ((size_t)n_vis + (size_t)n_text));
  w.partial = align64(w.minmax + rows * (size_t)(nvc + ntc) * 2);
  size_t end = align64(w.partial + rows * (size_t)(nvc + ntc) * (size_t)(d + 2));
  w.total_bytes = (end * sizeof(float) + 255) / 256 * 256;
  if (w.total_bytes == 0) w.total_bytes = 256;
  return w;
}

struct Calib {
  int mode;
  float tau1, tau2, gamma, delta;
};

// Compute units of the current device (cached per device; 256, the MI355X count, when there is
// no device, as in host-only checks of the plans).
long long device_cu_count();

// ---- launchers (each returns the hipError_t of its launches) -----------------------
hipError_t launch_quantize_generic(const void* x_f16, const cq_qtensor_t& out, int rows,
                                   int n_vis, int d, int bits, int axis, int group,
                                   hipStream_t stream);

// n_text_dev (all decode launchers): NULL, or a device int32 holding the current tail length; the
// kernels then attend to min(max(*n_text_dev, 0), s.n_text) text tokens.
hipError_t launch_decode_generic(const DecodeShape& s, const void* q, const cq_qtensor_t& k,
                                 const cq_qtensor_t& v, const void* k_text, const void* v_text,
                                 const int32_t* n_text_dev, const Calib& calib,
                                 float softmax_scale, void* out, float* workspace,
                                 const Workspace& wl, hipStream_t stream);

// First stage of the shape-agnostic decode on its own: raw logits [B*Hq][n_vis + n_text] and the
// extrema [B*Hq][n_chunks][2] of every chunk of tokens.
hipError_t launch_scores_generic(const DecodeShape& s, const void* q, const cq_qtensor_t& k,
                                 const void* k_text, const int32_t* n_text_dev,
                                 float softmax_scale, float* logits, float* minmax,
                                 hipStream_t stream);

// Grid search of the calibration parameters (Sec. 3.2): workspace layout in floats, and launcher.
constexpr int kMaxTauPairs = 64;
struct TauWorkspace {
  size_t logits_q;   // [B*Hq][n_vis + n_text]  logits on the dequantized keys and the text keys
  size_t logits_x;   // [B*Hq][n_vis]           logits on the exact 16-bit keys
  size_t minmax_q;   // [B*Hq][chunks of n_vis + chunks of n_text][2]
  size_t minmax_x;   // [B*Hq][chunks of n_vis][2]
  size_t sums;       // doubles: [n_pairs][B*Hq] and, with several chunks, [3 n_pairs + 2][B*Hq][n_chunks]
  int n_chunks;      // chunks per query row of the grid kernel
  size_t total_bytes;
  size_t reserve_bytes;   // the most that a tail of up to n_text tokens needs (never falls with n_text)
};
inline TauWorkspace tau_workspace_layout(int B, int Hq, int n_vis, int n_text, int n_pairs) {
  TauWorkspace w;
  // extrema of whichever logits kernels run: chunks of kVisChunk / kTextChunk tokens (the exact keys
  // go through the text-tail path), or at most kMaxTileChunks chunks
  auto most = [](int a) { return a > kMaxTileChunks ? a : kMaxTileChunks; };
  const int nvc = most(ceil_div(n_vis, kVisChunk)), ntc = most(ceil_div(n_text, kTextChunk));
  const int nxc = most(ceil_div(n_vis, kTextChunk));
  const size_t rows = (size_t)B * (size_t)Hq;
  // The size is that of 2 n_pairs + 1 sums for each of about four blocks per CU, blocks of whole rounds of one token
  // per thread: what a pass for the normalizers and one for the differences took, and what callers have reserved.  The
  // one pass has 3 n_pairs + 2 sums per chunk and takes as many chunks as fit.  With 4 x 4 pairs, long rows and from 128 rows on
  // these are 512 to 1023 blocks, two of which fill a CU, and 342 to 511 (a row each) where three shares of scratch hold one
  // chunk.  Against the two passes still 1.14 to 1.66 times as fast, 1 to 1500 rows x 1024 to 65536 tokens; 344, 400 and 480 rows
  // x 8192: 92.4 / 71.9, 98.8 / 75.7, 116 / 85.5 us.
  const int want = (int)((1024 + rows - 1) / rows), rounds = ceil_div(n_vis + n_text, 256);
  const int shares = rounds > 0 ? ceil_div(rounds, ceil_div(rounds, want)) : 1;
  const int fit = (shares * (2 * n_pairs + 1) - n_pairs) / (3 * n_pairs + 2);
  w.n_chunks = fit > 1 ? ceil_div(rounds, ceil_div(rounds, fit)) : 1;
  auto align64 = [](size_t x) { return (x + 63) / 64 * 64; };
  w.logits_q = 0;
  w.logits_x = align64(w.logits_q + rows * ((size_t)n_vis + (size_t)n_text));
  w.minmax_q = align64(w.logits_x + rows * (size_t)n_vis);
  w.minmax_x = align64(w.minmax_q + rows * (size_t)(nvc + ntc) * 2);
  w.sums = align64(w.minmax_x + rows * (size_t)nxc * 2);
  auto lay_out = [&](int n) {
    const size_t half = align64(w.sums + rows * (size_t)n * (size_t)(n_pairs + 1) * 2);
    const size_t end = align64(half + rows * (size_t)n * (size_t)n_pairs * 2);
    return (end * sizeof(float) + 255) / 256 * 256;
  };
  // whole rounds per chunk: one round more can mean fewer chunks, but never more than these
  w.reserve_bytes = lay_out(rounds > want ? want : rounds > 0 ? rounds : 1);
  w.total_bytes = lay_out(shares);
  return w;
}
hipError_t launch_tau_search(const DecodeShape& s, const void* q, const void* k_exact,
                             const cq_qtensor_t& k, const void* k_text, const float* tau1,
                             int n_tau1, const float* tau2, int n_tau2, float softmax_scale,
                             double* mse_out, float* workspace, const TauWorkspace& wl,
                             hipStream_t stream);

// Register-resident tile quantizer (quantize_tile.h): head_dim 64, 128 or 256, b in {1,2,4,8}, any
// channel-wise group of tokens, channel groups of 32 to 256, any n_vis, as far as a launch reaches.
bool quantize_tuned_supported(int rows, int n_vis, int d, int bits, int axis, int group);
bool quantize_tile_is_faster(int d, int bits, int axis, int group);
// One or two tensors of the same shape, in as few launches as their statistics allow.
struct QuantizeJob {
  const void* x_f16;
  cq_qtensor_t out;
  int axis, group;
};
hipError_t launch_quantize_tuned(const QuantizeJob* jobs, int n_jobs, int rows, int n_vis, int d, int bits,
                                 hipStream_t stream);
// its head dimensions other than 128
hipError_t launch_quantize_64(const QuantizeJob* jobs, int n_jobs, size_t n_tokens, int bits, hipStream_t stream);
hipError_t launch_quantize_256(const QuantizeJob* jobs, int n_jobs, size_t n_tokens, int bits, hipStream_t stream);

// Channel-wise groups that a workgroup's registers hold (quantize_slice.hip): one or two tensors with groups of the
// same size, in one launch.
bool quantize_slice_supported(size_t n_tokens, int d, int bits, int axis, int group);
hipError_t launch_quantize_slices(const QuantizeJob* jobs, int n_jobs, size_t n_tokens, int d, int bits, hipStream_t stream);

// Merge the per-chunk partials [n_rows][n_chunks][d + 2] of the online softmax into out.
hipError_t launch_combine(int n_rows, int n_chunks, int d, const float* partial, void* out,
                          hipStream_t stream);

// Rows that several workgroups of a launch share (decode_meet.h): how often a workgroup looks for the extrema of
// the others before it forms them itself.  A look takes about a third of a microsecond; workgroups whose
// neighbours start with the next round of a large grid wait for up to a round (50 us), and going on alone
// multiplies their work.  The bound (7 ms) is for a neighbour that never starts beside this one; calls that compete for the
// CUs do not come near it: 1, 2, 3 streams of calls of 512 workgroups, rows in 8 chunks, 19, 35, 52 us for a call of each
// (the mean of 200; the slowest 200 of 15: 21, 106, 123).
constexpr int kPatience = 20000;

// Tuned decode for head_dim 128 (see decode_fused.hip for the layouts it takes): one launch, a workgroup
// per row or per chunk of a row.  The plan is made once per call on the host and says what will run.
struct FusedPlan {
  bool ok = false;            // a tuned kernel exists for the shape
  int nhb = 1;                // blocks of 4 query heads per KV head
  int n_chunks = 1;           // chunks per row
  bool spread = false;        // every workgroup has a CU of its own, and as many chunks as pay
  bool fine = false;          // at the precision of the tile kernels (set by the caller; rows that end inside a group always are)
  bool ragged = false;        // rows that end inside a group
  int stride = 0;             // floats between the logit rows of two heads in LDS
  size_t lds = 0;             // dynamic LDS bytes per workgroup
  int patience = kPatience;
  size_t ws_partial_floats = 0;   // split rows: [counts | partials], offset in floats
  size_t ws_bytes = 256;      // workspace the launches touch (a multiple of 256, >= 256)
};
// min_chunks: 0 = as split says, n >= 1 = at least n (test override)
enum class FusedSplit {
  kWhole,    // whole rows where they fit on chip, else about the fewest chunks that do
  kFewest,   // exactly the fewest
  kSpread,   // more, where the chip has room for them
};
FusedPlan make_fused_plan(const DecodeShape& s, int min_chunks, FusedSplit split = FusedSplit::kWhole);
hipError_t launch_decode_fused(const DecodeShape& s, const FusedPlan& plan, const void* q,
                               const cq_qtensor_t& k, const cq_qtensor_t& v, const void* k_text,
                               const void* v_text, const int32_t* n_text_dev, const Calib& calib,
                               float softmax_scale, void* out, float* workspace,
                               hipStream_t stream);

// Streaming decode for split rows (decode_stream.hip): logits pass (all query heads of a KV head
// per workgroup, raw logits and chunk extrema to the workspace), values pass, combine.  Takes 1- and
// 2-bit codes, keys in groups of 128 tokens, token-wise values, up to 8 query heads per KV head.
struct StreamPlan {
  bool ok = false;
  int ca = 1, cb = 1;              // chunks per row of the logits pass / of the values pass
  int ct = 0;                      // chunks per row of the fp16 tail (values pass)
  size_t ws_lref_floats = 0;       // workspace: [extrema | group references | logits | partials],
  size_t ws_logits_floats = 0;     // offsets in floats
  size_t ws_partial_floats = 0;
  size_t ws_bytes = 256;
};
StreamPlan make_stream_plan(const DecodeShape& s, int min_chunks);
hipError_t launch_decode_stream(const DecodeShape& s, const StreamPlan& plan, const void* q,
                                const cq_qtensor_t& k, const cq_qtensor_t& v, const void* k_text,
                                const void* v_text, const int32_t* n_text_dev, const Calib& calib,
                                float softmax_scale, void* out, float* workspace,
                                hipStream_t stream);

// Tile decode (decode_tile.hip) for the layouts the two above do not take: head_dim 64, 128 or 256,
// channel-wise keys and values in groups of any size or values token-wise over the whole head, any
// number of query heads per KV head.  Logits pass, values pass, or both in one launch.
struct TilePlan {
  bool ok = false;
  int ca = 0, cb = 0;              // chunks per row of the visual tokens: logits pass, values pass
  int ct = 0, ct_tokens = 0;       // chunks per row of the fp16 tail, tokens per chunk
  size_t ws_minmax_floats = 0;     // workspace: [logits | extrema | partials | counts], offsets in floats
  size_t ws_partial_floats = 0, ws_count_floats = 0;
  // one launch instead of two, in a part of the same workspace: [words | counts | partials]
  bool one_launch = false;         // where the workgroups of a row exchange extrema
  bool one_launch_free = false;    // where they do not (no calibration, or a given range)
  int row_cb = 0, row_ct = 0;      // chunks per row of the visual tokens, of the tail
  size_t row_tags_floats = 0, row_partial_floats = 0;
  int patience = kPatience;
  size_t ws_bytes = 256;           // workspace the launches touch
  // the most that a tail of up to n_text tokens needs without a limit (never falls with n_text)
  size_t ws_reserve_bytes = 256;
};
// limit: the most scratch the plan may use; it takes fewer chunks to stay within it, and is not ok if
// one of each kind is still too much
TilePlan make_tile_plan(const DecodeShape& s, size_t limit = SIZE_MAX);
// The logits pass on its own, for keys of the same layouts whatever the values: raw logits
// [B*Hq][n_vis + n_text] and the extrema [B*Hq][ca + ct][2] of every chunk; in the same launch those of
// x_tokens 16-bit keys x_keys [B*Hkv][x_tokens][d], whose plan has them as a tail: [B*Hq][x_tokens] and
// [B*Hq][x_plan.ct][2].
TilePlan make_tile_logits_plan(const DecodeShape& s);
hipError_t launch_tile_logits(const DecodeShape& s, const TilePlan& plan, const void* q,
                              const cq_qtensor_t& k, const void* k_text, float softmax_scale,
                              float* logits, float* minmax, const TilePlan& x_plan, const void* x_keys,
                              int x_tokens, float* x_logits, float* x_minmax, hipStream_t stream);
hipError_t launch_decode_tile(const DecodeShape& s, const TilePlan& plan, const void* q,
                              const cq_qtensor_t& k, const cq_qtensor_t& v, const void* k_text,
                              const void* v_text, const int32_t* n_text_dev, const Calib& calib,
                              float softmax_scale, void* out, float* workspace, hipStream_t stream);

}  // namespace cq

#endif  // CQ_INTERNAL_H_
