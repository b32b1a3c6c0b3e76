// Grid search of the calibration parameters tau1, tau2 (Sec. 3.2).
//
// For every pair of the grid: the mean squared difference between the attention weights with the
// calibrated logits of the quantized keys, softmax([g(q K_deq^T s), q K_text^T s]), and the
// weights with the exact 16-bit keys, softmax([q K^T s, q K_text^T s]); mean over the attended
// tokens of a query row, then over all (batch, query head) rows.  gamma, delta of g are the
// extrema of the row's visual logits, as in the decode call.  The caller takes the argmin.
//
// A calibration-time utility, not part of the decode step: fp32 logits of both key sets (the tile
// kernels' logits pass where it takes the layout, else the shape-agnostic one; the exact keys pass
// as a 16-bit tail), the weights in fp64.
//
// The grid costs n1 + n2 + 2 exponentials per token (4 where the taus are evenly spaced from 0) instead of
// one per pair: with u = (s - gamma) / (delta - gamma),  g(s) = s + tau1 (u - 1) - tau2 u,  so a weight is
// e^s e^(tau1 (u - 1)) e^(-tau2 u).  Blocks of 4 x 4 pairs stay in registers; rows are cut into chunks
// where there are fewer than blocks that the chip holds (tau_workspace_layout has the number).
//
// One pass over the tokens.  With w and q the weights of the calibrated and of the exact keys before they are
// normalized, Z and Q their sums, the squared differences of the normalized ones need Z and Q, which are
// known only behind the last token.  But for any constant r of a row and pair, d = w - r q and S = sum d,
//     sum (w / Z - q / Q)^2 = (sum d^2 - 2 (S / Q) sum d q + (S / Q)^2 sum q^2) / Z^2,   Z = r Q + S,
// so three sums per pair and two per row, formed with Z and Q unknown, do.  r is the largest w (the largest q is
// 1): d is then as small as the difference that is asked for, equal weights give exactly 0, and
// what cancels in the bracket is the part of d along q only.
// Bound: fp64 arithmetic.  128 query rows x 3456 tokens, 4 x 4 grid: 416 us at first (one exponential
// per pair, a block per row), 55.6 us with factors and chunks, 42.8 with the sums folded by lane swaps,
// 32.9 with even spacing and the normalizers loaded eight at a time, 29.4 with both sets of logits in
// one launch (28.6 on another box), 20.2 in one pass instead of two (normalizers, then squared differences; 7.3 and
// 9.4 us of kernels).  Other sizes, two passes / one: 1 row x 256 + 8 tokens 14.1 / 10.8, 4096 x 2048 + 64 227 / 175, 1 row x 65536
// 35.2 / 30.8.
// The three sums per pair cost registers: 191 to 238 and two waves per SIMD (104 to 229 and two to four in the two passes),
// 9 to 97 scalar registers spilled (none with unevenly spaced factors).
// Against 64 bits 1e-8 to 8e-7, the same with one pass as with two: that is what the fp32 logits leave.
#include <cfloat>
#include <cmath>

#include "cq_internal.h"
#include "decode_fold.h"

namespace cq {
namespace {

constexpr int kThreads = 256;
constexpr int kGrid = 4;                 // pairs are taken 4 x 4 at a time
constexpr int kPairs = kGrid * kGrid;
// Largest |tau| whose factors e^(tau (u - 1)) and e^(-tau u) are formed on their own: products of the
// three factors then stay within e^+-150 of 1.  Beyond it every pair gets its own exponential.
constexpr double kFactorLimit = 50.0;

// How the weights of a block of pairs are formed.  kEven: both lists are evenly spaced (as {0, 1, 2, 3}
// is), so the factors of a list are a geometric series of two exponentials.
enum { kPairwise = 0, kFactors = 1, kEven = 2 };

struct TauArgs {
  float tau1[kMaxTauPairs], tau2[kMaxTauPairs];
  double step1, step2;                   // kEven: distance of neighbouring taus
  int n1, n2, n_vis, n_text, n_chunks, chunk_tokens;
  int ca, ct, cx;                        // chunk extrema: quantized visual, text, exact keys
  const float* logits_q;                 // [rows][n_vis + n_text]: quantized visual, then text
  const float* logits_x;                 // [rows][n_vis]: exact visual
  const float* minmax_q;                 // [rows][ca + ct][2]
  const float* minmax_x;                 // [rows][cx][2]
  size_t n_parts;                        // rows * n_chunks
  double* sums;                          // [3 n1 n2 + 2][rows][n_chunks]: S, sum d^2, sum d q per pair, then Q, sum q^2
  double* ratio;                         // [n1 n2][rows]: r;  one chunk per row: [rows][n1 n2] squared differences
};

// sum over each row of 16 lanes, every lane of the row gets it
__device__ inline double row_total(double v) {
  v += dpp_f64<0xB1>(v);      // quad_perm 1,0,3,2
  v += dpp_f64<0x4E>(v);      // quad_perm 2,3,0,1
  v += dpp_f64<0x141>(v);     // row_half_mirror
  return v + dpp_f64<0x140>(v);
}
__device__ inline double wave_total(double v) {
  v = row_total(v);
  v += __shfl_xor(v, 16);
  return v + __shfl_xor(v, 32);
}

// What every thread of a block knows about its query row.
struct Row {
  double gamma, inv_width, width, top_text, m_ref, m0;
};
__device__ inline Row row_extrema(const TauArgs& a, size_t row) {
  // the chunk extrema over the lanes of every wave
  const int lane = threadIdx.x & 63;
  float lo = FLT_MAX, hi = -FLT_MAX, tmax = -FLT_MAX, xmax = -FLT_MAX;
  const float* mq = a.minmax_q + row * (size_t)(a.ca + a.ct) * 2;
  for (int c = lane; c < a.ca; c += 64) {
    lo = fminf(lo, mq[2 * c]);
    hi = fmaxf(hi, mq[2 * c + 1]);
  }
  for (int c = lane; c < a.ct; c += 64) tmax = fmaxf(tmax, mq[2 * (a.ca + c) + 1]);
  const float* mx = a.minmax_x + row * (size_t)a.cx * 2;
  for (int c = lane; c < a.cx; c += 64) xmax = fmaxf(xmax, mx[2 * c + 1]);
  lo = row_min(lo);
  hi = row_max(hi);
  tmax = row_max(tmax);
  xmax = row_max(xmax);
#pragma unroll
  for (int o = 16; o <= 32; o <<= 1) {
    lo = fminf(lo, __shfl_xor(lo, o));
    hi = fmaxf(hi, __shfl_xor(hi, o));
    tmax = fmaxf(tmax, __shfl_xor(tmax, o));
    xmax = fmaxf(xmax, __shfl_xor(xmax, o));
  }
  Row r;
  r.gamma = lo;
  r.width = (double)hi - (double)lo;
  r.inv_width = r.width == 0.0 ? 0.0 : 1.0 / r.width;    // no range: slope 1, u = 0
  r.top_text = tmax;
  r.m_ref = fmax((double)xmax, (double)tmax);
  r.m0 = fmax((double)hi, (double)tmax);
  return r;
}

// The largest calibrated logit of a pair: g is monotone, so an end of [gamma, delta] or a text token has it.
__device__ inline double largest_logit(const Row& r, double tau1, double tau2) {
  const double at_lo = r.gamma - tau1;
  const double at_hi = r.width == 0.0 ? at_lo : r.gamma + r.width - tau2;
  return fmax(fmax(at_lo, at_hi), r.top_text);
}
__device__ inline double lane_value(double v, int lane) {      // wave-uniform copy of one lane's value
  const v2i x = __builtin_bit_cast(v2i, v);
  return __builtin_bit_cast(double, (v2i){__builtin_amdgcn_readlane(x[0], lane), __builtin_amdgcn_readlane(x[1], lane)});
}

// Weights (up to a factor per pair) of one token for the pairs (i0 + i, j0 + j), and of the exact keys.
// With factors: common reference m0 for all pairs.  Else pair by pair, with each pair's own reference,
// the largest calibrated logit.
template <int MODE>
__device__ inline void token_weights(const TauArgs& a, const Row& r, const double (&t1)[kGrid],
                                     const double (&t2)[kGrid], double s, double sx, bool vis,
                                     double (&w)[kPairs], double& ref) {
  ref = exp(sx - r.m_ref);
  const double u = (s - r.gamma) * r.inv_width;
  if constexpr (MODE != kPairwise) {
    const double e = exp(s - r.m0);
    double f1[kGrid], f2[kGrid];
    if constexpr (MODE == kEven) {
      const double x1 = vis ? u - 1.0 : 0.0, x2 = vis ? -u : 0.0;
      const double by1 = exp(a.step1 * x1), by2 = exp(a.step2 * x2);
      f1[0] = t1[0] == 0.0 ? e : e * exp(t1[0] * x1);          // wave-uniform
      f2[0] = t2[0] == 0.0 ? 1.0 : exp(t2[0] * x2);
#pragma unroll
      for (int i = 1; i < kGrid; ++i) {
        f1[i] = f1[i - 1] * by1;
        f2[i] = f2[i - 1] * by2;
      }
    } else {
#pragma unroll
      for (int i = 0; i < kGrid; ++i) {
        f1[i] = vis ? e * exp(t1[i] * (u - 1.0)) : e;
        f2[i] = vis ? exp(-t2[i] * u) : 1.0;
      }
    }
#pragma unroll
    for (int i = 0; i < kGrid; ++i)
#pragma unroll
      for (int j = 0; j < kGrid; ++j) w[i * kGrid + j] = f1[i] * f2[j];
  } else {
#pragma unroll
    for (int i = 0; i < kGrid; ++i)
#pragma unroll
      for (int j = 0; j < kGrid; ++j)
        w[i * kGrid + j] = exp((vis ? s + t1[i] * (u - 1.0) - t2[j] * u : s) - largest_logit(r, t1[i], t2[j]));
  }
}

// (sum d^2 - 2 (S / Q) sum d q + (S / Q)^2 sum q^2) / Z^2, see above; never below 0 by rounding, NaN stays NaN
__device__ inline double squared_difference(double S, double dd, double dq, double r, double Q, double qq) {
  const double Z = fma(r, Q, S), f = S / Q;
  const double v = fma(f, fma(f, qq, -2.0 * dq), dd) / (Z * Z);
  return v < 0.0 ? 0.0 : v;
}

// grid.x = rows * n_chunks.  ONE: a row is one chunk, whose block goes on to the squared differences.
template <int MODE, bool ONE>
__global__ void __launch_bounds__(kThreads)
tau_grid_kernel(const TauArgs a) {
  constexpr int kSums = 3 * kPairs + 2;
  __shared__ double red[kThreads / 64][kSums + 2];
  const size_t row = ONE ? blockIdx.x : blockIdx.x / (unsigned)a.n_chunks;
  const int chunk = ONE ? 0 : (int)(blockIdx.x - row * a.n_chunks);
  const int n_all = a.n_vis + a.n_text, n_pairs = a.n1 * a.n2;
  const int c0 = chunk * a.chunk_tokens, c1 = min(c0 + a.chunk_tokens, n_all);
  const float* sq = a.logits_q + row * (size_t)n_all;
  const float* sx = a.logits_x + row * (size_t)a.n_vis;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  auto logit_of = [&](int t) { return sq[min(t, n_all - 1)]; };
  auto exact_of = [&](int t) { return sx[min(t, a.n_vis - 1)]; };       // (of a text token: not used)
  const int t_first = c0 + (int)threadIdx.x;
  const float s_first = logit_of(t_first), x_first = exact_of(t_first); // asked for before the extrema are known
  const Row r = row_extrema(a, row);
  for (int i0 = 0; i0 < a.n1; i0 += kGrid)
    for (int j0 = 0; j0 < a.n2; j0 += kGrid) {
      double t1[kGrid], t2[kGrid], S[kPairs], dd[kPairs], dq[kPairs], Q = 0.0, qq = 0.0;
#pragma unroll
      for (int i = 0; i < kGrid; ++i) {        // beyond the grid: its last value again, not stored
        t1[i] = a.tau1[min(i0 + i, a.n1 - 1)];
        t2[i] = a.tau2[min(j0 + i, a.n2 - 1)];
      }
#pragma unroll
      for (int p = 0; p < kPairs; ++p) S[p] = dd[p] = dq[p] = 0.0;
      // the largest weight of pair lane % 16, then of every pair in scalar registers
      double own_ratio = 1.0, ratio[kPairs];
      if constexpr (MODE != kPairwise) {
        const double x1 = a.tau1[min(i0 + ((lane >> 2) & 3), a.n1 - 1)], x2 = a.tau2[min(j0 + (lane & 3), a.n2 - 1)];
        own_ratio = exp(largest_logit(r, x1, x2) - r.m0);
      }
#pragma unroll
      for (int p = 0; p < kPairs; ++p) ratio[p] = MODE == kPairwise ? 1.0 : lane_value(own_ratio, p);
      float s_next = s_first, x_next = x_first;
      for (int t = t_first; t < c1; t += kThreads) {
        const bool vis = t < a.n_vis;
        const double s = s_next, x = vis ? x_next : s_next;
        s_next = logit_of(t + kThreads);
        x_next = exact_of(t + kThreads);
        double w[kPairs], q;
        token_weights<MODE>(a, r, t1, t2, s, x, vis, w, q);
        Q += q;
        qq = fma(q, q, qq);
#pragma unroll
        for (int p = 0; p < kPairs; ++p) {
          const double d = fma(-ratio[p], q, w[p]);
          S[p] += d;
          dd[p] = fma(d, d, dd[p]);
          dq[p] = fma(d, q, dq[p]);
        }
      }
      __syncthreads();                         // the sums of the block of pairs before this one are out
      // four sums at a time: paired lane swaps leave one per row of 16 lanes (17 sums through LDS
      // exchanges took a third of the kernel)
      auto fold = [&](int at, double v0, double v1, double v2, double v3) {
        const double v = row_total(fold_rows(fold_halves(v0, v2), fold_halves(v1, v3)));
        if ((lane & 15) == 0) red[wave][at + (lane >> 4)] = v;
      };
#pragma unroll
      for (int p = 0; p < kPairs; p += 4) {
        fold(p, S[p], S[p + 1], S[p + 2], S[p + 3]);
        fold(kPairs + p, dd[p], dd[p + 1], dd[p + 2], dd[p + 3]);
        fold(2 * kPairs + p, dq[p], dq[p + 1], dq[p + 2], dq[p + 3]);
      }
      fold(3 * kPairs, Q, qq, 0.0, 0.0);
      __syncthreads();
      auto total = [&](int e) {
        double v = 0.0;
#pragma unroll
        for (int wv = 0; wv < kThreads / 64; ++wv) v += red[wv][e];
        return v;
      };
      const int e = threadIdx.x, p = e % kPairs, i = i0 + p / kGrid, j = j0 + p % kGrid;
      const bool exists = i < a.n1 && j < a.n2;
      if constexpr (ONE) {
        if (e < kPairs && exists)
          a.ratio[row * n_pairs + i * a.n2 + j] = squared_difference(total(p), total(kPairs + p), total(2 * kPairs + p), own_ratio,
                                                                     total(3 * kPairs), total(3 * kPairs + 1));
      } else {
        const size_t at = row * a.n_chunks + chunk;
        if (e < 3 * kPairs) {
          if (exists) a.sums[((size_t)(e / kPairs) * n_pairs + i * a.n2 + j) * a.n_parts + at] = total(e);
          if (e < kPairs && exists && chunk == 0) a.ratio[(size_t)(i * a.n2 + j) * (a.n_parts / a.n_chunks) + row] = own_ratio;
        } else if (e < kSums) {
          a.sums[((size_t)3 * n_pairs + (e - 3 * kPairs)) * a.n_parts + at] = total(e);
        }
      }
    }
}

// One block per pair: the squared differences of all rows, in a fixed order.  A thread takes a row: with one row of 65536 tokens
// one thread reads 129 chunks, 14 of that call's 31 us (2.0 us with 128 rows of 4 chunks).
template <bool ONE>
__global__ void __launch_bounds__(kThreads)
tau_reduce_kernel(const TauArgs a, size_t rows, double n_terms, double* __restrict__ mse_out) {
  __shared__ double red[kThreads / 64];
  const int n_pairs = a.n1 * a.n2, pair = blockIdx.x;
  double acc = 0.0;
  for (size_t r = threadIdx.x; r < rows; r += kThreads) {
    if constexpr (ONE) {
      acc += a.ratio[r * n_pairs + pair];
    } else {
      const size_t of[5] = {(size_t)pair, (size_t)n_pairs + pair, 2 * (size_t)n_pairs + pair, 3 * (size_t)n_pairs,
                            3 * (size_t)n_pairs + 1};
      double sum[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
      const double ratio = a.ratio[(size_t)pair * rows + r];
      for (int c0 = 0; c0 < a.n_chunks; c0 += 4) {             // twenty loads in flight
        double v[5][4];
#pragma unroll
        for (int k = 0; k < 5; ++k)
#pragma unroll
          for (int c = 0; c < 4; ++c) v[k][c] = a.sums[of[k] * a.n_parts + r * a.n_chunks + min(c0 + c, a.n_chunks - 1)];
#pragma unroll
        for (int k = 0; k < 5; ++k)
#pragma unroll
          for (int c = 0; c < 4; ++c) sum[k] += c0 + c < a.n_chunks ? v[k][c] : 0.0;
      }
      acc += squared_difference(sum[0], sum[1], sum[2], ratio, sum[3], sum[4]);
    }
  }
  acc = wave_total(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double v = 0.0;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) v += red[w];
    mse_out[pair] = v / n_terms;
  }
}

}  // namespace

hipError_t launch_tau_search(const DecodeShape& s, const void* q, const void* k_exact,
                             const cq_qtensor_t& k, const void* k_text, const float* tau1,
                             int n_tau1, const float* tau2, int n_tau2, float softmax_scale,
                             double* mse_out, float* workspace, const TauWorkspace& wl,
                             hipStream_t stream) {
  const size_t rows = (size_t)s.B * s.Hq;
  const int n_pairs = n_tau1 * n_tau2, n_all = s.n_vis + s.n_text;
  if (rows * wl.n_chunks > 0x7fffffffu || n_pairs > kMaxTauPairs) return hipErrorInvalidConfiguration;
  TauArgs a{};
  float* logits_q = workspace + wl.logits_q;
  float* logits_x = workspace + wl.logits_x;
  float* minmax_q = workspace + wl.minmax_q;
  float* minmax_x = workspace + wl.minmax_x;
  // logits on the quantized keys plus the text tail, then on the exact keys, which pass as a 16-bit
  // tail of n_vis tokens
  DecodeShape x = s;
  x.n_vis = 0;
  x.n_text = s.n_vis;
  x.n_text_cap = s.n_vis;
  x.n_vis_chunks = 0;
  x.n_text_chunks = ceil_div(s.n_vis, kTextChunk);
  x.n_chunks = x.n_text_chunks;
  static const cq_qtensor_t kNone = {nullptr, nullptr, nullptr};
  const TilePlan pq = make_tile_logits_plan(s), px = make_tile_logits_plan(x);
  if (pq.ok && px.ok) {
    a.ca = pq.ca; a.ct = pq.ct; a.cx = px.ct;
    const hipError_t e = launch_tile_logits(s, pq, q, k, k_text, softmax_scale, logits_q, minmax_q, px, k_exact,
                                            s.n_vis, logits_x, minmax_x, stream);
    if (e != hipSuccess) return e;
  } else {
    a.ca = s.n_vis_chunks; a.ct = s.n_text_chunks; a.cx = x.n_chunks;
    hipError_t e = launch_scores_generic(s, q, k, k_text, nullptr, softmax_scale, logits_q, minmax_q, stream);
    if (e != hipSuccess) return e;
    e = launch_scores_generic(x, q, kNone, k_exact, nullptr, softmax_scale, logits_x, minmax_x, stream);
    if (e != hipSuccess) return e;
  }
  a.n1 = n_tau1; a.n2 = n_tau2;
  bool factored = true;
  for (int i = 0; i < n_tau1; ++i) { a.tau1[i] = tau1[i]; factored = factored && std::fabs((double)tau1[i]) <= kFactorLimit; }
  for (int i = 0; i < n_tau2; ++i) { a.tau2[i] = tau2[i]; factored = factored && std::fabs((double)tau2[i]) <= kFactorLimit; }
  a.n_vis = s.n_vis; a.n_text = s.n_text;
  a.n_chunks = wl.n_chunks;
  a.chunk_tokens = ceil_div(ceil_div(n_all, kThreads), wl.n_chunks) * kThreads;
  a.logits_q = logits_q; a.logits_x = logits_x;
  a.minmax_q = minmax_q; a.minmax_x = minmax_x;
  a.n_parts = rows * wl.n_chunks;
  a.ratio = reinterpret_cast<double*>(workspace + wl.sums);
  a.sums = a.ratio + rows * n_pairs;
  const dim3 grid((unsigned)(rows * wl.n_chunks)), block(kThreads);
  auto spacing = [](const float* t, int n, double* step) {     // whether t is evenly spaced, exactly
    *step = n > 1 ? (double)t[1] - (double)t[0] : 0.0;
    for (int i = 2; i < n; ++i)
      if ((double)t[i] - (double)t[i - 1] != *step) return false;
    return true;
  };
  const bool even = spacing(tau1, n_tau1, &a.step1) && spacing(tau2, n_tau2, &a.step2);
  const int mode = !factored ? kPairwise : even ? kEven : kFactors;
  using GridKernel = void (*)(const TauArgs);
  static const GridKernel kern[3][2] = {{tau_grid_kernel<kPairwise, false>, tau_grid_kernel<kPairwise, true>},
                                        {tau_grid_kernel<kFactors, false>, tau_grid_kernel<kFactors, true>},
                                        {tau_grid_kernel<kEven, false>, tau_grid_kernel<kEven, true>}};
  const bool one = wl.n_chunks == 1;
  kern[mode][one]<<<grid, block, 0, stream>>>(a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  (one ? tau_reduce_kernel<true> : tau_reduce_kernel<false>)<<<dim3((unsigned)n_pairs), block, 0, stream>>>(
      a, rows, (double)n_all * (double)rows, mse_out);
  return hipGetLastError();
}

}  // namespace cq
