// Host side of libcq: argument validation, kernel-path selection, status strings.
// Every check here runs before the first HIP call, so a rejected call launches nothing.
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>

#include "cq_internal.h"
#include "decode_meet.h"

namespace cq {

u64 meeting_tag() {
  // a counter, mixed (the finalizer of splitmix64), from a start that differs between processes
  static std::atomic<u64> calls{(u64)std::chrono::steady_clock::now().time_since_epoch().count()};
  for (;;) {
    u64 z = calls.fetch_add(0x9e3779b97f4a7c15ull, std::memory_order_relaxed);
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    z = (z ^ (z >> 31)) & ~(u64)0xff;
    if ((unsigned)z != 0 && (unsigned)(z >> 32) != 0) return z;
  }
}

}  // namespace cq

namespace {

thread_local char g_last_error[256] = "";
// test / benchmark switches (cq_bench.h): per thread, never touched by the product calls
thread_local int g_kernel_path = CQ_PATH_AUTO;
thread_local int g_decode_chunks = 0;
thread_local bool g_alone = false, g_one_launch = false;

int fail(int status, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_last_error, sizeof(g_last_error), fmt, ap);
  va_end(ap);
  return status;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int check_group(const char* which, int axis, int group, int n_vis, int d) {
  if (axis == CQ_AXIS_CHANNEL) {
    if (group < 1) return fail(CQ_ERR_SHAPE, "%s_group must be >= 1 (got %d)", which, group);
    if (n_vis % group != 0)
      return fail(CQ_ERR_SHAPE, "n_vis=%d is not a multiple of %s_group=%d", n_vis, which, group);
  } else if (axis == CQ_AXIS_TOKEN) {
    if (group < 32 || group % 32 != 0 || d % group != 0)
      return fail(CQ_ERR_SHAPE,
                  "%s_group=%d must be a multiple of 32 that divides head_dim=%d", which, group, d);
  } else {
    return fail(CQ_ERR_UNSUPPORTED, "%s_axis=%d is not a CQ_AXIS_* value", which, axis);
  }
  return CQ_OK;
}

int check_layout(const cq_layout_t* L, bool need_q_heads, bool need_values = true) {
  if (!L) return fail(CQ_ERR_NULL, "layout is NULL");
  if (L->batch < 1 || L->n_kv_heads < 1)
    return fail(CQ_ERR_SHAPE, "batch=%d and n_kv_heads=%d must be >= 1", L->batch, L->n_kv_heads);
  if (need_q_heads && (L->n_q_heads < 1 || L->n_q_heads % L->n_kv_heads != 0))
    return fail(CQ_ERR_SHAPE, "n_q_heads=%d must be a positive multiple of n_kv_heads=%d",
                L->n_q_heads, L->n_kv_heads);
  if (L->head_dim < 32 || L->head_dim > 256 || L->head_dim % 32 != 0)
    return fail(CQ_ERR_SHAPE, "head_dim=%d must be a multiple of 32 in [32, 256]", L->head_dim);
  if (L->n_vis < 0) return fail(CQ_ERR_SHAPE, "n_vis=%d must be >= 0", L->n_vis);
  if (L->bits != 1 && L->bits != 2 && L->bits != 4 && L->bits != 8)
    return fail(CQ_ERR_UNSUPPORTED, "bits=%d not in {1, 2, 4, 8}", L->bits);
  int rc = check_group("k", L->k_axis, L->k_group, L->n_vis, L->head_dim);
  if (rc != CQ_OK) return rc;
  if (need_values) {
    rc = check_group("v", L->v_axis, L->v_group, L->n_vis, L->head_dim);
    if (rc != CQ_OK) return rc;
  }
  const double elems = (double)L->batch * L->n_kv_heads * (double)L->n_vis * L->head_dim;
  if (elems >= 9.0e18) return fail(CQ_ERR_SHAPE, "tensor too large");
  return CQ_OK;
}

int check_qtensor(const char* which, const cq_qtensor_t* t) {
  if (!t) return fail(CQ_ERR_NULL, "%s is NULL", which);
  if (!t->codes || !t->scale || !t->min)
    return fail(CQ_ERR_NULL, "%s has a NULL codes/scale/min pointer", which);
  if (!aligned16(t->codes) || !aligned16(t->scale) || !aligned16(t->min))
    return fail(CQ_ERR_ALIGN, "%s buffers must be 16-byte aligned", which);
  return CQ_OK;
}

cq::DecodeShape make_shape(const cq_layout_t* L, int n_text, int n_text_cap) {
  cq::DecodeShape s;
  s.B = L->batch; s.Hq = L->n_q_heads; s.Hkv = L->n_kv_heads; s.g = s.Hq / s.Hkv;
  s.d = L->head_dim; s.n_vis = L->n_vis; s.n_text = n_text; s.n_text_cap = n_text_cap;
  s.bits = L->bits; s.k_axis = L->k_axis; s.v_axis = L->v_axis;
  s.k_group = L->k_group; s.v_group = L->v_group;
  s.n_vis_chunks = cq::ceil_div(s.n_vis, cq::kVisChunk);
  s.n_text_chunks = cq::ceil_div(s.n_text, cq::kTextChunk);
  s.n_chunks = s.n_vis_chunks + s.n_text_chunks;
  s.words_per_token = s.d * s.bits / 32;
  return s;
}

int hip_fail(hipError_t e, const char* what) {
  return fail(CQ_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

}  // namespace

namespace {
// one new token per (batch, KV head) row into slot n_text of the fp16 tails: 16 bytes per thread
__global__ void __launch_bounds__(256) append_text_kernel(uint4* k_text, uint4* v_text, const uint4* k_new,
                                                          const uint4* v_new, int rows, int n_text,
                                                          int n_text_cap, int vec_per_token) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= rows * vec_per_token) return;
  const int row = i / vec_per_token, c = i % vec_per_token;
  const size_t dst = ((size_t)row * n_text_cap + n_text) * vec_per_token + c;
  k_text[dst] = k_new[i];
  v_text[dst] = v_new[i];
}
// The same with the tail length in device memory.  Nobody may raise the length before everybody has
// read it.  A step small enough for one workgroup with one piece of each tensor per thread copies,
// meets and raises it in one launch; a larger one is copied by many workgroups and the length raised by
// a launch of its own behind them.  Recorded in a graph, 8 KV heads of 128 channels: 1 to 8 sequences
// 3.4-3.6 us in two launches, 1.8 in one; 16 sequences 3.6 in two, 3.5 with two pieces per thread; 32
// sequences 3.6 in two, 8.1 with four (one CU waits for the address translation of every row).
constexpr int kAppendOneGroup = 1024;          // 16-byte pieces per tensor
__global__ void __launch_bounds__(kAppendOneGroup) append_text_step_kernel(uint4* k_text, uint4* v_text,
                                                                           const uint4* k_new, const uint4* v_new,
                                                                           int n, int32_t* n_text_dev,
                                                                           int n_text_cap, int vec_per_token) {
  const int i = threadIdx.x, j = min(i, n - 1);
  const uint4 k = k_new[j], v = v_new[j];                   // asked for before the length is known
  const int n_text = *n_text_dev;
  if (n_text < 0 || n_text >= n_text_cap) return;          // full tail: nothing is written
  if (i < n) {
    const int row = i / vec_per_token, c = i - row * vec_per_token;
    const size_t dst = ((size_t)row * n_text_cap + n_text) * vec_per_token + c;
    k_text[dst] = k;
    v_text[dst] = v;
  }
  __syncthreads();                                          // every thread has read the length
  if (i == 0) *n_text_dev = n_text + 1;
}
__global__ void __launch_bounds__(256) append_text_devlen_kernel(uint4* k_text, uint4* v_text, const uint4* k_new,
                                                                 const uint4* v_new, int rows,
                                                                 const int32_t* n_text_dev, int n_text_cap,
                                                                 int vec_per_token) {
  const int n_text = *n_text_dev;
  if (n_text < 0 || n_text >= n_text_cap) return;          // full tail: nothing is written
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= rows * vec_per_token) return;
  const int row = i / vec_per_token, c = i % vec_per_token;
  const size_t dst = ((size_t)row * n_text_cap + n_text) * vec_per_token + c;
  k_text[dst] = k_new[i];
  v_text[dst] = v_new[i];
}
__global__ void bump_tail_length_kernel(int32_t* n_text_dev, int n_text_cap) {
  const int n = *n_text_dev;
  if (n >= 0 && n < n_text_cap) *n_text_dev = n + 1;
}

// Everything cq_decode_attn* checks and decides on the host before the first HIP call.
struct DecodeCall {
  cq::DecodeShape shape;
  cq::Calib calib;
  float softmax_scale;
  bool tuned;               // a layout of the tuned kernels (else of the shape-agnostic ones)
  bool streamed;            // tuned, split rows: the streaming kernels with logits kept in scratch
  bool tiled;               // the tile kernels run, in place of either
  bool sets_fit;            // two head sets whose rows fit a workgroup each: the fused kernel can run, without scratch
  cq::FusedPlan plan;       // valid when tuned
  cq::StreamPlan stream;    // valid when streamed
  cq::TilePlan tile;        // valid when tiled
  cq::Workspace generic_ws;
  size_t ws_bytes;          // scratch the selected kernels touch
  size_t ws_query_bytes;    // scratch that serves this tail length and every shorter one
};

int check_calib(const cq_calib_t* calib, cq::Calib* c) {
  *c = cq::Calib{CQ_CALIB_NONE, 0.f, 0.f, 0.f, 0.f};
  if (!calib) return CQ_OK;
  if (calib->mode != CQ_CALIB_NONE && calib->mode != CQ_CALIB_DYNAMIC && calib->mode != CQ_CALIB_FIXED)
    return fail(CQ_ERR_UNSUPPORTED, "calib mode %d is not a CQ_CALIB_* value", calib->mode);
  c->mode = calib->mode;
  if (c->mode != CQ_CALIB_NONE) {
    if (!std::isfinite(calib->tau1) || !std::isfinite(calib->tau2))
      return fail(CQ_ERR_SHAPE, "tau1 and tau2 must be finite");
    c->tau1 = calib->tau1;
    c->tau2 = calib->tau2;
  }
  if (c->mode == CQ_CALIB_FIXED) {
    if (!std::isfinite(calib->gamma) || !std::isfinite(calib->delta) || !(calib->delta > calib->gamma))
      return fail(CQ_ERR_SHAPE, "CQ_CALIB_FIXED needs finite delta > gamma");
    c->gamma = calib->gamma;
    c->delta = calib->delta;
  }
  return CQ_OK;
}

// Two sets of query heads: visual tokens from which their whole rows stay on chip (see select_kernels).  Below, calls with
// many rows would lose: 256 rows x 128 + 100 tokens, 8 heads 12.7 us on the other kernels, 13.6 on chip.
constexpr int kTwoSetsOnChip = 256;

// Whether the tile kernels finish a call sooner than the tuned kernels that could take it on whole rows or the fewest
// chunks.  Decides where the fused kernel does not spread its rows over the chip (8 bits, two head sets of few
// tokens, more rows than CUs); of the calls that it does spread, says which would be the tile kernels' and keep their
// precision (select_kernels).  The fused kernel gives a row (a chunk of a row) to one CU, which moves about
// 27 GB/s, and the streaming kernels take three launches; with few rows the tile kernels, one or two launches
// over many small workgroups, win.  Microseconds per call inside a recorded graph, fitted to measurements of both sides
// (two launches of the tile kernels) over 8 to 256 rows (batch x KV heads) of 1024 to 32768 tokens, 1 to
// 8 bits, key groups of 32 tokens to the whole row, 1 to 6 query heads per KV head, none of them spread (the streaming
// kernels with two head sets: below 2 million tokens; longer rows have on_chip_is_faster, rows of more than one
// round whole_sets_are_faster); for example (tuned / tile)
//   1 bit, 4 heads:  8 rows x 3328 tokens 12.5 / 11.8, x 8192 21.8 / 14.4; 32 rows x 8192 22.1 / 19.6;
//                    8 rows x 1024 9.1 / 11.6 and 64 rows x 8192 22.2 / 27.1 stay fused
//   1 bit, 6 heads:  8 rows x 3328 20.7 / 12.5, 64 rows 22.6 / 19.5; 128 rows 26.0 / 27.3 stay streamed
//   4 bits:          32 rows x 3328 17.7 / 14.8;  8 bits: 8 rows x 3328 37.5 / 14.9, 16 x 10240 25.5 / 19.5
// The tail plays a part in one place: the streaming kernels read it once for two head sets, the tile
// kernels once for each (112 rows x 128 tokens, 8 heads, 1000 tail tokens: 23.4 / 28.9).  Over 700 drawn
// layouts of 1 to 500 rows with the tile kernels in two launches, 3 of the 285 that go to them are slower
// there by more than 2 %, the worst by 8 %; one launch is taken only where it is faster still.
bool tile_is_faster(cq::DecodeShape s, const cq::FusedPlan& with_tail) {
  const double rows = (double)s.B * s.Hkv, kn = s.n_vis * 1e-3, mtok = rows * s.n_vis * 1e-6;
  if (mtok > 2.0) return false;
  const double tail_k = rows * s.n_text * 1e-3;
  s.n_text = 0;
  const cq::FusedPlan plan = with_tail.n_chunks == 1 ? with_tail : cq::make_fused_plan(s, 0);
  const bool streamed = (plan.n_chunks > 1 || plan.nhb > 1) && cq::make_stream_plan(s, 0).ok;
  constexpr double kCus = 256.0;                                 // the whole chip, which all this is fitted to
  // bits:                           1     2     4     8
  static const double kTilePerM[] = {26.0, 28.0, 36.0, 58.0};    // per million tokens
  static const double kRowPerK[] = {1.65, 2.1, 3.0, 9.0};        // fused: per thousand tokens of a row
  const int i = s.bits == 1 ? 0 : s.bits == 2 ? 1 : s.bits == 4 ? 2 : 3;
  const bool two_sets = s.g > 4;
  const double tile = 10.6 + (two_sets ? 0.35 : 0.25) * kn + (two_sets ? 1.6 : 1.0) * kTilePerM[i] * mtok +
                      (two_sets && streamed ? 0.08 * tail_k : 0.0);
  const double group = s.k_axis == CQ_AXIS_CHANNEL && s.k_group == 32 ? 1.65 : s.k_group == 64 ? 1.25 : 1.0;
  const double per_k = kRowPerK[i] * group;
  const double workgroups = rows * plan.nhb * plan.n_chunks;
  const double rounds = std::ceil(workgroups / kCus), chunk_kn = kn / plan.n_chunks;
  const double tuned = plan.n_chunks == 1 && plan.nhb == 1 ? (s.bits == 8 ? 9.5 : 7.0) + per_k * kn * rounds
                       : streamed ? (two_sets ? 18.0 + 16.0 * mtok : 15.5 + 14.5 * mtok)
                                  : 12.0 + 1.5 * per_k * chunk_kn * rounds;
  return tile < 0.98 * tuned;
}

// Whether rows too long for one workgroup finish sooner in chunks of the fused kernel than on the streaming kernels, where
// the chunks take several rounds over the chip.  Microseconds, from 19 measured layouts of 18 to 320 rows x 9 to 63
// thousand tokens (streaming / fused): 4 heads, 1 bit, 144 rows x 10496 36.4 / 30.0, 100 x 21376 44.1 / 33.8; 2 bits,
// 64 x 55296 79.3 / 61.4; 7 heads 30 x 48128 54.2 / 39.7; but 8 heads, 216 rows x 18816 99 / 114 and 6 heads, 64 x 65536
// 81 / 100: six rounds, four rounds, and the streaming kernels expand the codes once for both head sets.  A
// tail that is half of the bytes counts too: 272 rows x 9088 + 830 in three rounds 55 / 63.
bool on_chip_is_faster(const cq::DecodeShape& s, const cq::FusedPlan& plan) {
  const double rows = (double)s.B * s.Hkv, mtok = rows * s.n_vis * 1e-6, c = plan.n_chunks;
  const double rounds = std::ceil(rows * plan.nhb * c / 256.0);
  const double chunk = (s.bits == 1 ? 1.6 : 2.1) * 1e-3 * s.n_vis / c + 0.9 * std::ceil(cq::ceil_div(s.n_text, 64) / c);
  const double fused = 7.8 + 1.25 * rounds * (chunk + 1.3);
  const double streamed = plan.nhb > 1 ? 38.0 + 11.0 * mtok : 15.5 + 14.5 * mtok;
  return fused < streamed;
}

// The same for two head sets whose rows fit a workgroup each: one launch that shares a row's lines through an XCD's L2 but reads
// the tail twice, in rounds over the chip, against three that read it once.  One round is always faster (64 rows x 3328
// tokens, 6 heads: 12.0 / 22.9 us).  Beyond, microseconds fitted to 28 measured layouts of 136 to 512 rows x 256 to
// 4608 + 31 to 1000 tokens (3 and 5 % rms; on chip / streaming): 224 rows x 768 + 38, 2 bits 15.6 / 22.3; 512 x 3328 + 128
// 46.2 / 60.9; but 512 x 256 + 1000 89.1 / 73.8, 424 x 768 + 804 76.9 / 56.0.  Three of the 28 go to the slower one, by 1, 2
// and 7 %.
bool whole_sets_are_faster(const cq::DecodeShape& s, const cq::FusedPlan& plan) {
  const double rows = (double)s.B * s.Hkv, rounds = std::ceil(rows * plan.nhb / 256.0);
  if (rounds <= 1.0 || !cq::make_stream_plan(s, 0).ok) return true;
  const double on_chip = -1.9 + rounds * (6.0 + (s.bits == 1 ? 1.3 : 1.7) * 1e-3 * s.n_vis + 1.0 * cq::ceil_div(s.n_text, 64));
  const double streamed = 15.1 + 24.6e-6 * rows * s.n_vis + 101e-6 * rows * s.n_text;
  return on_chip < streamed;
}

// Whether the tile kernels finish a call sooner than the fused kernel on rows with compute units to themselves, spread over them or
// whole: short rows with a long tail, which the chunks of a row share (each has four waves for it) while the tile kernels
// give it workgroups of its own.  Microseconds, fitted to 56 layouts of 1 to 83 rows x 157 to 4516 + 8 to 991 tokens (5 and
// 8 % rms; tile / fused): 8 rows x 446 + 511, 2 bits 9.4 / 12.5; 4 x 214 + 460, 4 bits 9.0 / 12.5; 8 x 1372 + 971, 2
// bits 11.4 / 13.2; but 40 x 846 + 902 19.2 / 15.4, 44 x 2304 + 160 13.5 / 11.2.  By less than 7 % neither is sure: of the
// layouts at issue two stay 2 % slower than they could be, and none moves to the slower side.
bool tiles_beat_spread_rows(const cq::DecodeShape& s, const cq::FusedPlan& plan) {
  const double rows = (double)s.B * s.Hkv, kn = s.n_vis * 1e-3, c = plan.n_chunks, sets = s.g > 4 ? 2.0 : 1.0;
  const int i = s.bits == 1 ? 0 : s.bits == 2 ? 1 : 2;
  static const double kTilePerM[] = {25.0, 27.0, 34.5}, kRowPerK[] = {1.35, 1.75, 2.6};
  const double group = s.k_axis == CQ_AXIS_CHANNEL && s.k_group == 32 ? 0.85 : 0.0;
  const double tile = 9.1 + 0.57 * kn + (sets > 1 ? 1.6 : 1.0) * kTilePerM[i] * rows * kn * 1e-3 +
                      0.104e-3 * sets * rows * s.n_text + (sets > 1 ? 0.3 : 0.0);
  const double fused = 5.1 + (c > 1 ? 3.8 + 0.05 * c : 0.0) + (kRowPerK[i] + group) * kn / c +
                       0.96 * std::ceil(cq::ceil_div(s.n_text, 64) / c) + 1.7 * rows * plan.nhb * c / 256.0;
  return tile < 0.93 * fused;
}

// Scratch of the kernels that run where the tile kernels do not.
size_t ws_without_tiles(const DecodeCall& c) {
  return c.streamed ? c.stream.ws_bytes : c.tuned ? c.plan.ws_bytes : c.generic_ws.total_bytes;
}

// Kernel selection and scratch size for a valid layout: one plan per call, used by the size query,
// by the argument check and by the launch.
// scratch_limit: the most scratch the caller can offer.  Rows that have to be split run on the
// streaming kernels, which keep the raw logits in scratch (2 bytes per query head and visual
// token); when that does not fit the limit they run as chunks of the fused kernel, whose logits stay on
// chip and which keeps only extrema and partials in scratch.
int select_kernels(const cq_layout_t* L, int n_text, int n_text_cap, size_t scratch_limit,
                   DecodeCall* call) {
  call->shape = make_shape(L, n_text, n_text_cap);
  call->plan = cq::make_fused_plan(call->shape, g_decode_chunks,
                                   g_kernel_path == CQ_PATH_AUTO ? cq::FusedSplit::kSpread : cq::FusedSplit::kWhole);
  if (g_alone) call->plan.patience = 0;
  if (g_kernel_path == CQ_PATH_TUNED && !call->plan.ok)
    return fail(CQ_ERR_UNSUPPORTED, "no tuned decode kernel for this layout");
  call->tuned = g_kernel_path != CQ_PATH_GENERIC && call->plan.ok;
  call->streamed = false;
  auto sets_fit = [&] {
    return call->plan.n_chunks == 1 && call->plan.nhb > 1 && L->n_vis >= kTwoSetsOnChip && L->bits <= 4 && g_decode_chunks == 0;
  };
  const bool whole_sets = sets_fit() && whole_sets_are_faster(call->shape, call->plan);
  bool on_chip = whole_sets || (call->plan.spread && (call->plan.nhb == 1 || L->n_vis >= kTwoSetsOnChip));
  // Calls that stay here instead of going to the tile kernels keep the precision of those, or go there.
  bool to_tiles = false;
  if (on_chip && g_kernel_path == CQ_PATH_AUTO) {
    const cq::FusedPlan rows = call->plan.n_chunks == 1 ? call->plan : cq::make_fused_plan(call->shape, 0);
    if (call->plan.ragged || tile_is_faster(call->shape, rows)) {
      to_tiles = call->plan.spread && tiles_beat_spread_rows(call->shape, call->plan);
      call->plan.fine = !to_tiles;
      if (to_tiles) {
        call->plan = rows;
        on_chip = false;
      }
    }
  }
  call->sets_fit = sets_fit();
  size_t reserve = 0;                // scratch that shorter tails may use on other kernels
  if (call->tuned && (call->plan.n_chunks > 1 || call->plan.nhb > 1) && !g_one_launch && !on_chip) {
    call->stream = cq::make_stream_plan(call->shape, g_decode_chunks);
    if (call->stream.ok && g_kernel_path == CQ_PATH_AUTO && g_decode_chunks == 0 && call->plan.n_chunks > 1 &&
        on_chip_is_faster(call->shape, call->plan)) {
      on_chip = true;
      reserve = call->stream.ws_bytes;
    } else {
      call->streamed = call->stream.ok && call->stream.ws_bytes <= scratch_limit;
    }
  }
  call->generic_ws = cq::workspace_layout(L->batch, L->n_q_heads, L->head_dim, L->n_vis, n_text);
  call->tiled = false;
  // Every entry point runs the same kernels on a layout that the tuned ones do not take.  Where the
  // shape-agnostic kernels fit the scratch of the allocation-free entry point, the tile kernels stay
  // within it too, with fewer chunks if need be; where they would not, that entry point refuses
  // what does not fit.
  const size_t most = (size_t)CQ_NOALLOC_SCRATCH_BYTES;
  if (g_kernel_path == CQ_PATH_TILE) {
    call->tile = cq::make_tile_plan(call->shape);
    call->tiled = call->tile.ok;
    if (!call->tiled) return fail(CQ_ERR_UNSUPPORTED, "no tile decode kernel for this layout");
    reserve = call->tile.ws_reserve_bytes;
  } else if (g_kernel_path == CQ_PATH_AUTO && !call->tuned) {
    const bool within = call->generic_ws.total_bytes <= most;
    call->tile = cq::make_tile_plan(call->shape, within ? most : SIZE_MAX);
    call->tiled = call->tile.ok && call->tile.ws_bytes <= scratch_limit;
    reserve = within && call->tile.ws_reserve_bytes > most ? most : call->tiled ? call->tile.ws_reserve_bytes : 0;
  } else if (g_kernel_path == CQ_PATH_AUTO && L->n_vis > 0 && g_decode_chunks == 0 && !on_chip) {
    cq::DecodeShape no_tail = call->shape;
    no_tail.n_text = 0;
    const bool faster = to_tiles || tile_is_faster(call->shape, call->plan);
    if (faster || (no_tail.g > 4 && tile_is_faster(no_tail, call->plan))) {
      // Not beyond the scratch of the allocation-free entry point: both entry points run the same kernels.
      // By the size that never falls as the tail grows: where a tail stays here, so does every shorter one.
      call->tile = cq::make_tile_plan(call->shape);
      call->tiled = faster && call->tile.ok && call->tile.ws_reserve_bytes <= most;
      if (call->tiled || (call->tile.ok && cq::make_tile_plan(no_tail).ws_reserve_bytes <= most))
        reserve = call->tile.ws_reserve_bytes < most ? call->tile.ws_reserve_bytes : most;
    }
  }
  if (g_alone) call->tile.patience = 0;
  call->ws_bytes = call->tiled ? call->tile.ws_bytes : ws_without_tiles(*call);
  call->ws_query_bytes = reserve > call->ws_bytes ? reserve : call->ws_bytes;
  return CQ_OK;
}

// Argument checks of cq_decode_attn, cq_decode_attn_devlen and the allocation-free variant;
// n_text is the tail length or (n_text_dev != NULL) the host's bound of it.
int check_decode(const cq_layout_t* L, const void* q_f16, const cq_qtensor_t* k,
                 const cq_qtensor_t* v, const void* k_text_f16, const void* v_text_f16,
                 int32_t n_text, int32_t n_text_cap, bool length_on_device,
                 const cq_calib_t* calib, float softmax_scale, const void* out_f16,
                 size_t scratch_limit, DecodeCall* call) {
  int rc = check_layout(L, true);
  if (rc != CQ_OK) return rc;
  if (!q_f16 || !out_f16) return fail(CQ_ERR_NULL, "q_f16 or out_f16 is NULL");
  if (!aligned16(q_f16) || !aligned16(out_f16))
    return fail(CQ_ERR_ALIGN, "q_f16 and out_f16 must be 16-byte aligned");
  if (n_text < 0 || n_text_cap < n_text)
    return fail(CQ_ERR_SHAPE, "need 0 <= n_text (%d) <= n_text_cap (%d)", n_text, n_text_cap);
  if ((long long)L->n_vis + n_text < 1)
    return fail(CQ_ERR_SHAPE, "nothing to attend to: n_vis + n_text == 0");
  if (L->n_vis > 0) {
    if ((rc = check_qtensor("k", k)) != CQ_OK) return rc;
    if ((rc = check_qtensor("v", v)) != CQ_OK) return rc;
  }
  if (n_text > 0 || (length_on_device && n_text_cap > 0)) {
    if (n_text > 0 && (!k_text_f16 || !v_text_f16))
      return fail(CQ_ERR_NULL, "n_text=%d but k_text_f16 or v_text_f16 is NULL", n_text);
    if (!aligned16(k_text_f16) || !aligned16(v_text_f16))
      return fail(CQ_ERR_ALIGN, "text-tail tensors must be 16-byte aligned");
  }
  if ((rc = check_calib(calib, &call->calib)) != CQ_OK) return rc;
  if (!std::isfinite(softmax_scale) || softmax_scale < 0.f)
    return fail(CQ_ERR_SHAPE, "softmax_scale must be finite and >= 0");
  call->softmax_scale = softmax_scale == 0.f ? 1.0f / std::sqrt((float)L->head_dim) : softmax_scale;
  return select_kernels(L, n_text, n_text_cap, scratch_limit, call);
}

int launch_decode(const DecodeCall& call, const void* q_f16, const cq_qtensor_t* k,
                  const cq_qtensor_t* v, const void* k_text_f16, const void* v_text_f16,
                  const int32_t* n_text_dev, void* out_f16, void* workspace, void* stream) {
  static const cq_qtensor_t kNone = {nullptr, nullptr, nullptr};
  const cq_qtensor_t& kq = k ? *k : kNone;
  const cq_qtensor_t& vq = v ? *v : kNone;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const hipError_t e = call.tiled
      ? cq::launch_decode_tile(call.shape, call.tile, q_f16, kq, vq, k_text_f16, v_text_f16,
                               n_text_dev, call.calib, call.softmax_scale, out_f16,
                               static_cast<float*>(workspace), st)
      : call.streamed
      ? cq::launch_decode_stream(call.shape, call.stream, q_f16, kq, vq, k_text_f16, v_text_f16,
                                 n_text_dev, call.calib, call.softmax_scale, out_f16,
                                 static_cast<float*>(workspace), st)
      : call.tuned
      ? cq::launch_decode_fused(call.shape, call.plan, q_f16, kq, vq, k_text_f16, v_text_f16,
                                n_text_dev, call.calib, call.softmax_scale, out_f16,
                                static_cast<float*>(workspace), st)
      : cq::launch_decode_generic(call.shape, q_f16, kq, vq, k_text_f16, v_text_f16, n_text_dev,
                                  call.calib, call.softmax_scale, out_f16,
                                  static_cast<float*>(workspace), call.generic_ws, st);
  if (e != hipSuccess) return hip_fail(e, "decode attention");
  return CQ_OK;
}

// Scratch of the allocation-free entry point: part of the library's device image, so every GPU the
// library runs on holds its own copy at its own address until the process ends.  On the host
// this name is only a handle for hipGetSymbolAddress, never an address: kernels and copies get
// the pointer that noalloc_scratch() returns.
static __device__ __align__(256) unsigned char scratch[CQ_NOALLOC_SCRATCH_BYTES];
constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch_ptr[kMaxDevices];

// Device address of `scratch` on the current device, looked up once per device.
int noalloc_scratch(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  if (dev < 0 || dev >= kMaxDevices) return fail(CQ_ERR_HIP, "device index %d is out of range", dev);
  void* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (!p) {
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
    if (!p || (reinterpret_cast<uintptr_t>(p) & 255u) != 0)
      return fail(CQ_ERR_HIP, "the scratch array has no 256-byte aligned device address");
    g_scratch_ptr[dev].store(p, std::memory_order_release);   // same value from every thread
  }
  *out = p;
  return CQ_OK;
}

// The kernels that the tile kernels stand in for need less scratch (256 bytes where one workgroup owns
// a row), and so does the fused kernel in place of the streaming ones: a workspace that holds what they need,
// but not more, is accepted, and they run.
int check_workspace(DecodeCall* call, const void* workspace, size_t workspace_bytes) {
  if (!workspace) return fail(CQ_ERR_WORKSPACE, "workspace is NULL");
  if ((reinterpret_cast<uintptr_t>(workspace) & 255u) != 0)
    return fail(CQ_ERR_WORKSPACE, "workspace must be 256-byte aligned");
  if (call->streamed && call->sets_fit && g_kernel_path == CQ_PATH_AUTO && workspace_bytes < call->stream.ws_bytes &&
      workspace_bytes >= call->plan.ws_bytes) {
    call->streamed = false;
    if (!call->tiled) call->ws_bytes = ws_without_tiles(*call);
  }
  if (call->tiled && g_kernel_path == CQ_PATH_AUTO && workspace_bytes < call->ws_bytes &&
      workspace_bytes >= ws_without_tiles(*call)) {
    call->tiled = false;
    call->ws_bytes = ws_without_tiles(*call);
  }
  // Rows of the fused kernel in more chunks than they must be (to fill the chip, or with a shorter tail the last round
  // of workgroups) than the workspace holds partials of: the fewest that fit on chip, which never grow as
  // the tail shrinks.
  if (call->tuned && !call->streamed && !call->tiled && call->plan.n_chunks > 1 && workspace_bytes < call->ws_bytes &&
      g_decode_chunks == 0) {
    const cq::FusedPlan fewest = cq::make_fused_plan(call->shape, 0, cq::FusedSplit::kFewest);
    if (fewest.ok && fewest.ws_bytes <= workspace_bytes) {
      call->plan = fewest;
      call->ws_bytes = fewest.ws_bytes;
    }
  }
  if (workspace_bytes < call->ws_bytes)
    return fail(CQ_ERR_WORKSPACE, "workspace has %zu bytes, %zu needed", workspace_bytes, call->ws_bytes);
  return CQ_OK;
}

}  // namespace

extern "C" {

int cq_version(void) { return 200; }

const char* cq_last_error(void) { return g_last_error; }

const char* cq_status_string(int status) {
  switch (status) {
    case CQ_OK: return "CQ_OK";
    case CQ_ERR_NULL: return "CQ_ERR_NULL: a required pointer is NULL";
    case CQ_ERR_SHAPE: return "CQ_ERR_SHAPE: sizes out of range or not divisible";
    case CQ_ERR_UNSUPPORTED: return "CQ_ERR_UNSUPPORTED: bits, axis or group not supported";
    case CQ_ERR_WORKSPACE: return "CQ_ERR_WORKSPACE: workspace missing, misaligned or too small";
    case CQ_ERR_HIP: return "CQ_ERR_HIP: a HIP call or kernel launch failed";
    case CQ_ERR_ALIGN: return "CQ_ERR_ALIGN: a tensor pointer is not 16-byte aligned";
    default: return "unknown cq_status";
  }
}

int cq_bench_set_kernel_path(int path) {
  if (path < CQ_PATH_AUTO || path > CQ_PATH_TILE)
    return fail(CQ_ERR_UNSUPPORTED, "unknown kernel path %d", path);
  const int prev = g_kernel_path;
  g_kernel_path = path;
  return prev;
}

int cq_bench_set_decode_chunks(int n_chunks) {
  if (n_chunks < 0) return fail(CQ_ERR_SHAPE, "n_chunks=%d must be >= 0", n_chunks);
  const int prev = g_decode_chunks + (g_alone ? CQ_CHUNKS_ALONE : 0) + (g_one_launch ? CQ_CHUNKS_ONE_LAUNCH : 0);
  g_alone = n_chunks & CQ_CHUNKS_ALONE;
  g_one_launch = n_chunks & CQ_CHUNKS_ONE_LAUNCH;
  g_decode_chunks = n_chunks & (CQ_CHUNKS_ALONE - 1);
  return prev;
}

size_t cq_decode_workspace_bytes(const cq_layout_t* L, int32_t n_text, const cq_calib_t* calib) {
  cq::Calib c;
  if (check_layout(L, true) != CQ_OK || n_text < 0 || check_calib(calib, &c) != CQ_OK) return 0;
  DecodeCall call;
  if (select_kernels(L, n_text, n_text, SIZE_MAX, &call) != CQ_OK) return 0;
  return call.ws_query_bytes;
}

int cq_quantize_kv(const cq_layout_t* L, const void* k_f16, const void* v_f16,
                   const cq_qtensor_t* k_out, const cq_qtensor_t* v_out, void* stream) {
  int rc = check_layout(L, false);
  if (rc != CQ_OK) return rc;
  const bool do_k = (k_f16 != nullptr) || (k_out != nullptr);
  const bool do_v = (v_f16 != nullptr) || (v_out != nullptr);
  if (!do_k && !do_v) return fail(CQ_ERR_NULL, "both the key and the value pair are NULL");
  if (do_k) {
    if (!k_f16) return fail(CQ_ERR_NULL, "k_f16 is NULL but k_out is not");
    if ((rc = check_qtensor("k_out", k_out)) != CQ_OK) return rc;
    if (!aligned16(k_f16)) return fail(CQ_ERR_ALIGN, "k_f16 must be 16-byte aligned");
  }
  if (do_v) {
    if (!v_f16) return fail(CQ_ERR_NULL, "v_f16 is NULL but v_out is not");
    if ((rc = check_qtensor("v_out", v_out)) != CQ_OK) return rc;
    if (!aligned16(v_f16)) return fail(CQ_ERR_ALIGN, "v_f16 must be 16-byte aligned");
  }
  if (L->n_vis == 0) return CQ_OK;
  const int path = g_kernel_path == CQ_PATH_TILE ? CQ_PATH_TUNED : g_kernel_path, rows = L->batch * L->n_kv_heads;
  const bool k_tuned = cq::quantize_tuned_supported(rows, L->n_vis, L->head_dim, L->bits, L->k_axis, L->k_group);
  const bool v_tuned = cq::quantize_tuned_supported(rows, L->n_vis, L->head_dim, L->bits, L->v_axis, L->v_group);
  if (path == CQ_PATH_TUNED && ((do_k && !k_tuned) || (do_v && !v_tuned)))
    return fail(CQ_ERR_UNSUPPORTED, "no tuned quantizer for this layout");
  hipStream_t s = static_cast<hipStream_t>(stream);
  cq::QuantizeJob jobs[2];         // tensors that the tile kernels take, together
  int n_jobs = 0;
  for (int i = 0; i < 2; ++i) {
    if (i == 0 ? !do_k : !do_v) continue;
    const cq::QuantizeJob job = i == 0 ? cq::QuantizeJob{k_f16, *k_out, L->k_axis, L->k_group}
                                       : cq::QuantizeJob{v_f16, *v_out, L->v_axis, L->v_group};
    if (path != CQ_PATH_GENERIC && (i == 0 ? k_tuned : v_tuned) &&
        (path == CQ_PATH_TUNED || cq::quantize_tile_is_faster(L->head_dim, L->bits, job.axis, job.group))) {
      jobs[n_jobs++] = job;
      continue;
    }
    const hipError_t e = cq::launch_quantize_generic(job.x_f16, job.out, rows, L->n_vis, L->head_dim, L->bits,
                                                     job.axis, job.group, s);
    if (e != hipSuccess) return hip_fail(e, i == 0 ? "quantize keys" : "quantize values");
  }
  if (n_jobs > 0) {
    const hipError_t e = cq::launch_quantize_tuned(jobs, n_jobs, rows, L->n_vis, L->head_dim, L->bits, s);
    if (e != hipSuccess) return hip_fail(e, "quantize");
  }
  return CQ_OK;
}

int cq_decode_attn(const cq_layout_t* L, const void* q_f16, const cq_qtensor_t* k,
                   const cq_qtensor_t* v, const void* k_text_f16, const void* v_text_f16,
                   int32_t n_text, int32_t n_text_cap, const cq_calib_t* calib,
                   float softmax_scale, void* out_f16, void* workspace, size_t workspace_bytes,
                   void* stream) {
  DecodeCall call;
  int rc = check_decode(L, q_f16, k, v, k_text_f16, v_text_f16, n_text, n_text_cap, false, calib,
                        softmax_scale, out_f16, SIZE_MAX, &call);
  if (rc != CQ_OK) return rc;
  if ((rc = check_workspace(&call, workspace, workspace_bytes)) != CQ_OK) return rc;
  return launch_decode(call, q_f16, k, v, k_text_f16, v_text_f16, nullptr, out_f16, workspace, stream);
}

int cq_decode_attn_noalloc(const cq_layout_t* L, const void* q_f16, const cq_qtensor_t* k,
                           const cq_qtensor_t* v, const void* k_text_f16, const void* v_text_f16,
                           int32_t n_text, int32_t n_text_cap, const cq_calib_t* calib,
                           float softmax_scale, void* out_f16, void* stream) {
  DecodeCall call;
  int rc = check_decode(L, q_f16, k, v, k_text_f16, v_text_f16, n_text, n_text_cap, false, calib,
                        softmax_scale, out_f16, (size_t)CQ_NOALLOC_SCRATCH_BYTES, &call);
  if (rc != CQ_OK) return rc;
  if (call.ws_bytes > (size_t)CQ_NOALLOC_SCRATCH_BYTES)
    return fail(CQ_ERR_WORKSPACE,
                "this shape needs %zu bytes of scratch, the allocation-free entry point holds %zu: "
                "call cq_decode_attn with a workspace", call.ws_bytes,
                (size_t)CQ_NOALLOC_SCRATCH_BYTES);
  void* ws = nullptr;
  if ((rc = noalloc_scratch(&ws)) != CQ_OK) return rc;
  return launch_decode(call, q_f16, k, v, k_text_f16, v_text_f16, nullptr, out_f16, ws, stream);
}

int cq_decode_attn_devlen(const cq_layout_t* L, const void* q_f16, const cq_qtensor_t* k,
                          const cq_qtensor_t* v, const void* k_text_f16, const void* v_text_f16,
                          const int32_t* n_text_dev, int32_t n_text_max, int32_t n_text_cap,
                          const cq_calib_t* calib, float softmax_scale, void* out_f16,
                          void* workspace, size_t workspace_bytes, void* stream) {
  if (!n_text_dev) return fail(CQ_ERR_NULL, "n_text_dev is NULL");
  if ((reinterpret_cast<uintptr_t>(n_text_dev) & 3u) != 0)
    return fail(CQ_ERR_ALIGN, "n_text_dev must be 4-byte aligned");
  DecodeCall call;
  int rc = check_decode(L, q_f16, k, v, k_text_f16, v_text_f16, n_text_max, n_text_cap, true, calib,
                        softmax_scale, out_f16, SIZE_MAX, &call);
  if (rc != CQ_OK) return rc;
  if ((rc = check_workspace(&call, workspace, workspace_bytes)) != CQ_OK) return rc;
  return launch_decode(call, q_f16, k, v, k_text_f16, v_text_f16, n_text_dev, out_f16, workspace,
                       stream);
}

size_t cq_tau_search_workspace_bytes(const cq_layout_t* L, int32_t n_text, int32_t n_tau1,
                                     int32_t n_tau2) {
  if (check_layout(L, true, false) != CQ_OK || n_text < 0 || n_tau1 < 1 || n_tau2 < 1 ||
      (long long)n_tau1 * n_tau2 > cq::kMaxTauPairs)
    return 0;
  return cq::tau_workspace_layout(L->batch, L->n_q_heads, L->n_vis, n_text, n_tau1 * n_tau2)
      .reserve_bytes;
}

int cq_tau_search(const cq_layout_t* L, const void* q_f16, const void* k_exact_f16,
                  const cq_qtensor_t* k, const void* k_text_f16, int32_t n_text, int32_t n_text_cap,
                  const float* tau1, int32_t n_tau1, const float* tau2, int32_t n_tau2,
                  float softmax_scale, double* mse_out, void* workspace, size_t workspace_bytes,
                  void* stream) {
  int rc = check_layout(L, true, false);     // the values play no part
  if (rc != CQ_OK) return rc;
  if (L->n_vis < 1) return fail(CQ_ERR_SHAPE, "no quantized tokens to calibrate: n_vis == 0");
  if (!q_f16 || !k_exact_f16 || !mse_out || !tau1 || !tau2)
    return fail(CQ_ERR_NULL, "q_f16, k_exact_f16, tau1, tau2 or mse_out is NULL");
  if (!aligned16(q_f16) || !aligned16(k_exact_f16))
    return fail(CQ_ERR_ALIGN, "q_f16 and k_exact_f16 must be 16-byte aligned");
  if ((reinterpret_cast<uintptr_t>(mse_out) & 7u) != 0)
    return fail(CQ_ERR_ALIGN, "mse_out must be 8-byte aligned");
  if ((rc = check_qtensor("k", k)) != CQ_OK) return rc;
  if (n_text < 0 || n_text_cap < n_text)
    return fail(CQ_ERR_SHAPE, "need 0 <= n_text (%d) <= n_text_cap (%d)", n_text, n_text_cap);
  if (n_text > 0) {
    if (!k_text_f16) return fail(CQ_ERR_NULL, "n_text=%d but k_text_f16 is NULL", n_text);
    if (!aligned16(k_text_f16)) return fail(CQ_ERR_ALIGN, "k_text_f16 must be 16-byte aligned");
  }
  if (n_tau1 < 1 || n_tau2 < 1 || (long long)n_tau1 * n_tau2 > cq::kMaxTauPairs)
    return fail(CQ_ERR_SHAPE, "the grid needs 1 <= n_tau1 * n_tau2 <= %d pairs (got %d x %d)",
                cq::kMaxTauPairs, n_tau1, n_tau2);
  for (int i = 0; i < n_tau1; ++i)
    if (!std::isfinite(tau1[i])) return fail(CQ_ERR_SHAPE, "tau1[%d] is not finite", i);
  for (int i = 0; i < n_tau2; ++i)
    if (!std::isfinite(tau2[i])) return fail(CQ_ERR_SHAPE, "tau2[%d] is not finite", i);
  if (!std::isfinite(softmax_scale) || softmax_scale < 0.f)
    return fail(CQ_ERR_SHAPE, "softmax_scale must be finite and >= 0");
  if (softmax_scale == 0.f) softmax_scale = 1.0f / std::sqrt((float)L->head_dim);
  const cq::TauWorkspace wl =
      cq::tau_workspace_layout(L->batch, L->n_q_heads, L->n_vis, n_text, n_tau1 * n_tau2);
  if (!workspace) return fail(CQ_ERR_WORKSPACE, "workspace is NULL");
  if ((reinterpret_cast<uintptr_t>(workspace) & 255u) != 0)
    return fail(CQ_ERR_WORKSPACE, "workspace must be 256-byte aligned");
  if (workspace_bytes < wl.total_bytes)
    return fail(CQ_ERR_WORKSPACE, "workspace has %zu bytes, %zu needed", workspace_bytes,
                wl.total_bytes);
  const cq::DecodeShape s = make_shape(L, n_text, n_text_cap);
  const hipError_t e = cq::launch_tau_search(s, q_f16, k_exact_f16, *k, k_text_f16, tau1, n_tau1,
                                             tau2, n_tau2, softmax_scale, mse_out,
                                             static_cast<float*>(workspace), wl,
                                             static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return hip_fail(e, "tau search");
  return CQ_OK;
}

static int check_append(const cq_layout_t* L, const void* k_text_f16, const void* v_text_f16,
                        int32_t n_text_cap, const void* k_new_f16, const void* v_new_f16,
                        long long* n_vec, int* vec_per_token) {
  int rc = check_layout(L, false);
  if (rc != CQ_OK) return rc;
  if (!k_text_f16 || !v_text_f16 || !k_new_f16 || !v_new_f16)
    return fail(CQ_ERR_NULL, "a tail or new-token pointer is NULL");
  if (!aligned16(k_text_f16) || !aligned16(v_text_f16) || !aligned16(k_new_f16) ||
      !aligned16(v_new_f16))
    return fail(CQ_ERR_ALIGN, "tails and new-token tensors must be 16-byte aligned");
  if (n_text_cap < 1) return fail(CQ_ERR_SHAPE, "the tail has no capacity: n_text_cap=%d", n_text_cap);
  const long long rows = (long long)L->batch * L->n_kv_heads;
  *vec_per_token = L->head_dim * 2 / 16;          // head_dim is a multiple of 32
  *n_vec = rows * *vec_per_token;
  if (*n_vec > 0x7fffffffLL) return fail(CQ_ERR_SHAPE, "batch * n_kv_heads * head_dim is too large");
  return CQ_OK;
}

int cq_append_text_kv(const cq_layout_t* L, void* k_text_f16, void* v_text_f16, int32_t n_text,
                      int32_t n_text_cap, const void* k_new_f16, const void* v_new_f16,
                      void* stream) {
  long long n;
  int vec_per_token;
  int rc = check_append(L, k_text_f16, v_text_f16, n_text_cap > 0 ? n_text_cap : 1, k_new_f16,
                        v_new_f16, &n, &vec_per_token);
  if (rc != CQ_OK) return rc;
  if (n_text < 0 || n_text >= n_text_cap)
    return fail(CQ_ERR_SHAPE, "the tail is full or n_text is negative: n_text=%d, n_text_cap=%d",
                n_text, n_text_cap);
  append_text_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0,
                       static_cast<hipStream_t>(stream)>>>(
      static_cast<uint4*>(k_text_f16), static_cast<uint4*>(v_text_f16),
      static_cast<const uint4*>(k_new_f16), static_cast<const uint4*>(v_new_f16),
      (int)(n / vec_per_token), n_text, n_text_cap, vec_per_token);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(CQ_ERR_HIP, "append_text_kernel: %s", hipGetErrorString(e));
  return CQ_OK;
}

int cq_append_text_kv_devlen(const cq_layout_t* L, void* k_text_f16, void* v_text_f16,
                             int32_t* n_text_dev, int32_t n_text_cap, const void* k_new_f16,
                             const void* v_new_f16, void* stream) {
  long long n;
  int vec_per_token;
  int rc = check_append(L, k_text_f16, v_text_f16, n_text_cap, k_new_f16, v_new_f16, &n,
                        &vec_per_token);
  if (rc != CQ_OK) return rc;
  if (!n_text_dev) return fail(CQ_ERR_NULL, "n_text_dev is NULL");
  if ((reinterpret_cast<uintptr_t>(n_text_dev) & 3u) != 0)
    return fail(CQ_ERR_ALIGN, "n_text_dev must be 4-byte aligned");
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (n <= kAppendOneGroup) {
    append_text_step_kernel<<<dim3(1), dim3((unsigned)((n + 63) / 64 * 64)), 0, st>>>(
        static_cast<uint4*>(k_text_f16), static_cast<uint4*>(v_text_f16), static_cast<const uint4*>(k_new_f16),
        static_cast<const uint4*>(v_new_f16), (int)n, n_text_dev, n_text_cap, vec_per_token);
    const hipError_t e1 = hipGetLastError();
    if (e1 != hipSuccess) return fail(CQ_ERR_HIP, "append_text_step_kernel: %s", hipGetErrorString(e1));
    return CQ_OK;
  }
  append_text_devlen_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st>>>(
      static_cast<uint4*>(k_text_f16), static_cast<uint4*>(v_text_f16),
      static_cast<const uint4*>(k_new_f16), static_cast<const uint4*>(v_new_f16),
      (int)(n / vec_per_token), n_text_dev, n_text_cap, vec_per_token);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(CQ_ERR_HIP, "append_text_devlen_kernel: %s", hipGetErrorString(e));
  bump_tail_length_kernel<<<dim3(1), dim3(1), 0, st>>>(n_text_dev, n_text_cap);
  e = hipGetLastError();
  if (e != hipSuccess) return fail(CQ_ERR_HIP, "bump_tail_length_kernel: %s", hipGetErrorString(e));
  return CQ_OK;
}

}  // extern "C"
