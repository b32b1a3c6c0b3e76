// Tile quantizer for head_dim 64, 128 and 256, b in {1, 2, 4, 8}, any group of tokens (channel axis)
// or of channels (token axis), any number of tokens (gfx950).  Included by quantize_tuned.hip,
// quantize_64.hip and quantize_256.hip, which instantiate it for their head dimensions.
//
// One 256-thread block quantizes a tile of 128 tokens x D channels (32 KB of fp16 at D = 128), read
// once with 16-byte loads and kept in registers:
//   lane = (token slot lane / (D/8), channel octet lane % (D/8)); wave w owns tokens 32w .. 32w+31,
//   so a wave-wide load is 512/D whole token rows = 1 KB contiguous.
//   1. min/max of Sec. 3.1 with packed-half min/max: over tokens (channel axis: in-thread, then
//      across the token slots and, for groups > 32 tokens, across waves through LDS) or over
//      channels (token axis: in-thread over the octet, then across the lanes of a channel group).
//   2. one thread per (group, channel) resp. (token, channel group) derives, in fp64 where every
//      quantity is exact, the stored scale/min and 2^b-1 fp16 thresholds t_k such that for every
//      fp16 x:  x > t_k  <=>  round-half-even((x-min)(2^b-1)/(max-min)) >= k   (Sec. 2.2 equation).
//   3. codes by comparing packed halves against the thresholds (sign of t - x), bits gathered with
//      v_perm + v_dot4, words assembled across adjacent lanes, MSB first as in the packing appendix.
//   b in {4, 8} (too many thresholds): step 2 stores min and (2^b-1)/(max-min) per group, step 3
//   evaluates the quantize equation per element with that reciprocal - in fp32 where that already
//   decides the code, in fp64 with the rounding settled exactly (see exact_code) where it does
//   not; a lane's 8 channels fill one word (b = 4) or two (b = 8).
//
// How tokens are dealt to tiles.  Statistics per token, and per channel over 32, 64 or 128 tokens, do
// not care where a row ends (the row is a whole number of groups), so all rows are one run of
// tokens cut every 128; only the very last tile can be short.  A short tile reads its last token
// again in place of the missing ones, which changes no extremum, and stores only what exists.
// Channel-wise groups of any other size are "whole" sequences of their own (Sec. 3.1 as printed
// when the group is n_vis).  Up to 128 tokens are one short tile; those that a workgroup's registers hold go to
// quantize_slice.hip.  Longer ones take a pass of their own: row_extrema_kernel leaves `splits` partial
// (min, max) pairs per channel in the code words of the sequence's LAST tile (the caller's output
// buffer: no other memory is needed), the tile kernel reduces them instead of computing tile statistics,
// and the last tile of every sequence is quantized by a second launch, after all other tiles have read
// the partials it overwrites.
// The FIRST tile of a sequence is the short one, so the last one always has room for the partials.
// Results are bit-identical to evaluating the quantize equation element by element in fp64.
//
// Bound: HBM, and the launches of a small call.  Groups of a few tokens spend a block on little
// (quantize_tile_is_faster has the line from which these kernels are used).  128 x 8
// rows x 16384 tokens, 1 bit, groups of 128 (9.33 GB): 1669 us = 5.6 TB/s.
#ifndef CQ_QUANTIZE_TILE_H_
#define CQ_QUANTIZE_TILE_H_

#include <hip/hip_fp16.h>

#include "cq_internal.h"

namespace cq {
namespace {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef _Float16 v4h __attribute__((ext_vector_type(4)));
typedef unsigned int v2u __attribute__((ext_vector_type(2)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));

constexpr int kTile = 128;       // tokens per block
constexpr int kThreads = 256;

// The value of lane ^ 1 (0xB1), lane ^ 2 (0x4E), of the half row mirrored (0x141) or the row (0x140), moved inside
// the vector unit; every lane of the wave is active.  A small call is one chain of such steps: with __shfl_xor, an
// LDS round trip each, 8 rows x 3328 tokens at 2 bits took 8.6 us, now 7.7 (large calls are HBM-bound: the same).
template <int CTRL>
__device__ inline uint32_t other_lane(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xF, 0xF, true);
}

// ---- fp16 bit patterns as an ordered set
__device__ inline uint16_t h_key(uint16_t u) { return (u & 0x8000u) ? (uint16_t)~u : (uint16_t)(u | 0x8000u); }
__device__ inline uint16_t h_unkey(uint16_t k) { return (k & 0x8000u) ? (uint16_t)(k & 0x7fffu) : (uint16_t)~k; }
__device__ inline uint16_t h_next(uint16_t u) { return h_unkey((uint16_t)(h_key(u) + 1)); }
__device__ inline uint16_t h_prev(uint16_t u) { return h_unkey((uint16_t)(h_key(u) - 1)); }
__device__ inline double h_to_double(uint16_t u) { return (double)__half2float(__ushort_as_half(u)); }

// Largest fp16 t (as bits) with  NOT [ 2L(t - alpha) ? (2k-1) D ],  ? being > for odd k and >= for
// even k (the even side of a tie).  Then code >= k  <=>  x > t for every fp16 x.
__device__ inline uint16_t threshold_bits(double alpha, double D, int k, int L) {
  if (!(D > 0.0)) return 0x7bffu;            // constant group: nothing exceeds the largest finite
  const double rhs = (double)(2 * k - 1) * D, twoL = 2.0 * L;
  const bool strict = (k & 1) != 0;
  auto pred = [&](uint16_t u) {
    const double lhs = twoL * (h_to_double(u) - alpha);
    return strict ? lhs > rhs : lhs >= rhs;
  };
  // candidate: the real-valued boundary, good to an fp16 step (the reciprocal of 2L is a compile-time
  // constant at every call site; the loops below make the result exact whatever the candidate)
  uint16_t t = __half_as_ushort(__float2half_rn((float)(alpha + rhs * (1.0 / twoL))));
  // (its neighbours are tried along with it, not one behind the other, each a chain of fp64 instructions and a branch)
  const uint16_t below = h_prev(t);
  const bool over = pred(t), over_below = pred(below), over_above = pred(h_next(t));
  if (over ? over_below : !over_above) {     // more than a step off
    for (int it = 0; it < 4 && pred(t); ++it) t = h_prev(t);
    for (int it = 0; it < 4 && !pred(h_next(t)); ++it) t = h_next(t);
  } else if (over) {
    t = below;
  }
  return t == 0x8000u ? (uint16_t)0 : t;     // -0 would break the sign test against +0
}

__device__ inline uint16_t canonical_zero(uint16_t bits) { return (bits & 0x7fffu) == 0 ? (uint16_t)0 : bits; }

// Extrema over the tokens of a wave whose lanes hold 8 channels each, STRIDE lanes to a token: lo[c], hi[c] of the
// wave's channels.  In the vector unit: lane rotations within a row of 16 lanes, then paired swaps of registers
// over halves and rows of the wave, each of which leaves half as many registers.  With LDS exchanges, eight registers at each
// distance, and the threshold's candidates one behind the other, 64 rows x 3003 tokens, 2 bits took 32.6 us, now 31.5; 80 x
// 3003 46.1 / 44.2; 64 rows x 2500 tokens of 256 channels, 1 bit 48.4 / 45.9.
template <int STRIDE>
__device__ inline void store_extrema(v8h mn, v8h mx, int lane, _Float16* lo, _Float16* hi) {
  v4u a = __builtin_bit_cast(v4u, mn), b = __builtin_bit_cast(v4u, mx);
  auto least = [](uint32_t x, uint32_t y) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(v2h, x), __builtin_bit_cast(v2h, y)));
  };
  auto most = [](uint32_t x, uint32_t y) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(v2h, x), __builtin_bit_cast(v2h, y)));
  };
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if constexpr (STRIDE <= 4) {
      a[r] = least(a[r], other_lane<0x124>(a[r]));           // row_ror 4
      b[r] = most(b[r], other_lane<0x124>(b[r]));
    }
    if constexpr (STRIDE <= 8) {
      a[r] = least(a[r], other_lane<0x128>(a[r]));           // row_ror 8
      b[r] = most(b[r], other_lane<0x128>(b[r]));
    }
  }
  // registers 0, 1 of the whole wave in lanes 0-31, registers 2, 3 in lanes 32-63
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const auto x = __builtin_amdgcn_permlane32_swap(a[r], a[r + 2], false, false);
    const auto y = __builtin_amdgcn_permlane32_swap(b[r], b[r + 2], false, false);
    a[r] = least(x[0], x[1]);
    b[r] = most(y[0], y[1]);
  }
  const int oct = lane & (STRIDE - 1);
  if constexpr (STRIDE == 32) {
    const int at = 8 * oct + 4 * (lane >> 5);
    *reinterpret_cast<v2u*>(lo + at) = (v2u){a[0], a[1]};
    *reinterpret_cast<v2u*>(hi + at) = (v2u){b[0], b[1]};
  } else {                                                   // register r in the r-th row of lanes
    const auto x = __builtin_amdgcn_permlane16_swap(a[0], a[1], false, false);
    const auto y = __builtin_amdgcn_permlane16_swap(b[0], b[1], false, false);
    if ((lane & 15) < STRIDE) {
      const int at = 8 * oct + 2 * (lane >> 4);
      *reinterpret_cast<uint32_t*>(lo + at) = least(x[0], x[1]);
      *reinterpret_cast<uint32_t*>(hi + at) = most(y[0], y[1]);
    }
  }
}

// t - x for 8 channels, two to a register: its sign bits say x > t.  (Written out because the compiler takes a packed
// subtraction apart, into two subtractions and a third instruction that joins them.)
__device__ inline v4u differences(const v8h& t, const v8h& x) {
  const v4u a = __builtin_bit_cast(v4u, t), b = __builtin_bit_cast(v4u, x);
  v4u d;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    unsigned v;
    asm("v_pk_add_f16 %0, %1, %2 neg_lo:[0,1] neg_hi:[0,1]" : "=v"(v) : "v"(a[r]), "v"(b[r]));
    d[r] = v;
  }
  return d;
}
// the sign bits of four 16-bit numbers as bytes, 0 or -1, first number in the low byte
__device__ inline int sign_bytes(uint32_t d01, uint32_t d23) { return (int)__builtin_amdgcn_perm(d23, d01, 0x0b0a0908u); }

// Code bits of one octet of one token: 8 bits (b = 1) or 16 bits (b = 2), first channel highest.  Four signs at a
// time become bits by a product of bytes whose other factors are minus the powers of two they stand for: 8 and 25
// instructions for the octet (19 and 56 with the differences as the compiler forms them, masks and unsigned products).
// us, before / now, keys and values: 64 rows x 3003 tokens, 2 bits, whole-sequence groups 36.0 / 32.6, 1 bit 27.7 / 26.2;
// 8 rows x 3328, 2 bits, groups of 128 7.8 / 7.2; 128 rows x 3328, 2 bits, groups of 32 50.3 / 45.8 (large calls of one bit are
// HBM-bound: the same).
template <int BITS>
__device__ inline uint32_t octet_codes(const v8h& x, const v8h* thr) {
  if constexpr (BITS == 1) {
    const v4u d = differences(thr[0], x);
    const int s = __builtin_amdgcn_sdot4(sign_bytes(d[0], d[1]), (int)0xf0e0c080u, 0, false);
    return (uint32_t)__builtin_amdgcn_sdot4(sign_bytes(d[2], d[3]), (int)0xfffefcf8u, s, false);
  } else {
    const v4u d2 = differences(thr[1], x);                   // high code bit: x > t2
    const v4u dl = differences(thr[0], x) ^ d2 ^ differences(thr[2], x);      // low one
    int s = __builtin_amdgcn_sdot4(sign_bytes(d2[0], d2[1]), (int)0xfef8e080u, 0, false);
    s = __builtin_amdgcn_sdot4(sign_bytes(dl[0], dl[1]), (int)0xfffcf0c0u, s, false);
    s = __builtin_amdgcn_sdot4(sign_bytes(d2[2], d2[3]), (int)0xfef8e080u, s << 8, false);
    return (uint32_t)__builtin_amdgcn_sdot4(sign_bytes(dl[2], dl[3]), (int)0xfffcf0c0u, s, false);
  }
}

// round-half-even((x - alpha) L / D) for b in {4, 8}, from rinv = fl(L / D) (0 for a constant group).
// x - alpha is exact in fp64; q = fl((x - alpha) * rinv) is within 2^-44 of the true quotient
// (two roundings, q <= 255).  The true quotient is a ratio of integers with denominator
// D / 2^-24 < 2^41, so it is either exactly k + 1/2 or at least 2^-42 away from it: a computed
// fraction within 2^-43 of 1/2 is a tie (to even), anything else rounds by its computed fraction.
__device__ inline uint32_t exact_code(_Float16 x, double alpha, double rinv) {
  const double q = ((double)(float)x - alpha) * rinv;
  const double f = floor(q);
  const double frac = q - f;
  uint32_t c = (uint32_t)(int)f;
  if (fabs(frac - 0.5) < 0x1p-43) c += c & 1u;
  else c += frac > 0.5 ? 1u : 0u;
  return c;
}

// the 8 codes of one octet as packed words, first channel in the top bits (packing appendix).
// Fast path in fp32 with alpha32 = alpha and rinv32 = fl32(rinv): q32 = fl(fl(x - alpha) * rinv32)
// carries three roundings, so it is within L * 3 * 2^-24 of the true quotient (L = 2^b - 1 bounds
// the quotient).  Unless q32 lies within L * 2^-22 of a half-integer, rounding it to nearest gives
// the exact code; an octet with any element inside that band (8-bit codes: ~0.1 % of the octets)
// is redone by exact_code.
template <int BITS>
__device__ inline void octet_words(const v8h& x, const double (&alpha)[8], const double (&rinv)[8],
                                   const float (&alpha32)[8], const float (&rinv32)[8],
                                   uint32_t& w0, uint32_t& w1) {
  constexpr float kBand = (float)((1 << BITS) - 1) * 0x1p-22f;
  uint32_t c[8];
  bool unsure = false;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const float q = ((float)x[j] - alpha32[j]) * rinv32[j];
    const float r = rintf(q);
    c[j] = (uint32_t)(int)r;
    unsure |= 0.5f - fabsf(q - r) <= kBand;
  }
  if (unsure) {
#pragma unroll
    for (int j = 0; j < 8; ++j) c[j] = exact_code(x[j], alpha[j], rinv[j]);
  }
  if constexpr (BITS == 4) {
    w0 = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) w0 |= c[j] << (28 - 4 * j);
    w1 = 0;
  } else {
    w0 = (c[0] << 24) | (c[1] << 16) | (c[2] << 8) | c[3];
    w1 = (c[4] << 24) | (c[5] << 16) | (c[6] << 8) | c[7];
  }
}

struct QArgs {
  const __half* x;
  uint32_t* codes;
  float* scale;
  uint16_t* minv;
  size_t n_tokens;         // tokens of all rows
  int tile_stride;         // tokens between tile starts: 128, or the group when it is one short tile
  // long groups only: tokens per group, tiles per group, tokens of the first tile, the tiles of every
  // group that this launch covers (tile_first .. tile_first + tiles_launch - 1), partial extrema
  int seq_tokens, tiles_seq, first_tokens, tile_first, tiles_launch, splits;
  unsigned launch_magic;   // fl(2^32 / tiles_launch) + 1 if exact for every block of the launch, else 0
};

// Most partial extrema that fit the code words of one tile: splits * 2 * D fp16 <= 128 * D * b / 8 bytes.
constexpr int max_splits(int bits) { return 4 * bits; }

// Partial extrema of a sequence's split sp live at [(sp * 2 + {0: min, 1: max}) * D + channel], fp16,
// in the code words of its last tile.
template <int D, int BITS>
__device__ inline _Float16* seq_partials(const QArgs& a, size_t seq) {
  const size_t last_tok = (seq + 1) * (size_t)a.seq_tokens - kTile;
  return reinterpret_cast<_Float16*>(a.codes + last_tok * (D * BITS / 32));
}

// First pass of a long group: block (sequence, sp) scans its share of the tokens.  The first n_first
// blocks work on one tensor, the rest on the other (as in the tile kernels below).
template <int D, int BITS>
__global__ void __launch_bounds__(kThreads)
row_extrema_kernel(const QArgs first, const QArgs second, unsigned n_first) {
  constexpr int kOct = D / 8, kSlots = 64 / kOct, kLoads = 32 / kSlots;
  __shared__ __align__(16) _Float16 s_part[2][4][D];
  const QArgs a = blockIdx.x < n_first ? first : second;
  const unsigned block = blockIdx.x < n_first ? blockIdx.x : blockIdx.x - n_first;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c8 = lane & (kOct - 1), ts = lane / kOct;
  const unsigned seq = block / (unsigned)a.splits, sp = block - seq * (unsigned)a.splits;
  const int t0 = (int)((long long)a.seq_tokens * sp / a.splits);
  const int t1 = (int)((long long)a.seq_tokens * (sp + 1) / a.splits);     // > t0: a share has tokens
  const v8h* src = reinterpret_cast<const v8h*>(a.x) + (size_t)seq * a.seq_tokens * kOct + c8;
  const _Float16 inf = __builtin_bit_cast(_Float16, (uint16_t)0x7c00u);
  v8h mn = {inf, inf, inf, inf, inf, inf, inf, inf};
  v8h mx = -mn;
  for (int t = t0; t < t1; t += kTile) {
    v8h x[kLoads];
#pragma unroll
    for (int i = 0; i < kLoads; ++i)           // past the share's end: its last token again
      x[i] = src[(size_t)min(t + 32 * wave + kSlots * i + ts, t1 - 1) * kOct];
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      mn = __builtin_elementwise_min(mn, x[i]);
      mx = __builtin_elementwise_max(mx, x[i]);
    }
  }
  store_extrema<kOct>(mn, mx, lane, s_part[0][wave], s_part[1][wave]);
  __syncthreads();
  if (tid < D) {
    _Float16 lo = s_part[0][0][tid], hi = s_part[1][0][tid];
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      lo = (_Float16)fminf((float)lo, (float)s_part[0][w][tid]);
      hi = (_Float16)fmaxf((float)hi, (float)s_part[1][w][tid]);
    }
    _Float16* part = seq_partials<D, BITS>(a, seq);
    part[(sp * 2 + 0) * D + tid] = lo;
    part[(sp * 2 + 1) * D + tid] = hi;
  }
}

// What a tile needs in LDS.
template <int D, int AXIS, int BITS, int GROUP>
struct TileMem {
  static constexpr int L = (1 << BITS) - 1;
  static constexpr int kG = GROUP == 0 ? kTile : GROUP;   // a tile of a long group is one group
  static constexpr int NG = AXIS == CQ_AXIS_CHANNEL ? kTile / kG : D / kG;          // groups per tile / token
  static constexpr bool kWide = BITS > 2;                 // per-element arithmetic instead of thresholds
  static constexpr int kPerTok = NG > 4 ? NG : 4;         // token axis: slots per token
  static constexpr int kStats = AXIS == CQ_AXIS_CHANNEL ? NG * D : kTile * kPerTok; // group slots of the tile
  __align__(16) _Float16 s_part[2][4][AXIS == CQ_AXIS_CHANNEL ? D : 8];   // per-wave min, max
  __align__(16) _Float16 s_stat[AXIS == CQ_AXIS_TOKEN ? kStats : 1][2];   // min, max
  __align__(16) _Float16 s_thr[kWide ? 8 : (AXIS == CQ_AXIS_CHANNEL ? NG * L * D : kStats * 4)];
  __align__(16) double s_rinv[kWide ? kStats : 1];
  __align__(16) _Float16 s_alpha[kWide ? kStats : 8];
  __align__(16) uint32_t s_codes[kTile * (D * BITS / 32)];
};

// AXIS: CQ_AXIS_CHANNEL (GROUP tokens per group; GROUP = 0: long groups, extrema from
// row_extrema_kernel) or CQ_AXIS_TOKEN (GROUP channels per group).  SHORT = false: the caller knows that
// every tile is full.
template <int D, int AXIS, int BITS, int GROUP, bool SHORT = true>
__device__ __forceinline__ void quantize_tile(const QArgs& a, const unsigned block, TileMem<D, AXIS, BITS, GROUP>& sm) {
  using Mem = TileMem<D, AXIS, BITS, GROUP>;
  constexpr int kOct = D / 8;                             // lanes per token
  constexpr int kSlots = 64 / kOct, kLoads = 32 / kSlots; // tokens per wave-wide load, loads per wave
  constexpr int L = Mem::L, kG = Mem::kG, NG = Mem::NG, kPerTok = Mem::kPerTok;
  constexpr int kWords = D * BITS / 32;                   // words per token
  constexpr bool kWhole = GROUP == 0, kWide = Mem::kWide;
  constexpr int kParts = BITS == 2 ? 2 : 1;               // threads per group slot in step 2, three thresholds shared: 8 rows x 3328, 7.1 / 6.7 us
  static_assert(!kWhole || AXIS == CQ_AXIS_CHANNEL, "long groups are channel-wise");
  auto& s_part = sm.s_part;
  auto& s_stat = sm.s_stat;
  auto& s_thr = sm.s_thr;
  auto& s_rinv = sm.s_rinv;
  auto& s_alpha = sm.s_alpha;
  auto& s_codes = sm.s_codes;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c8 = lane & (kOct - 1), ts = lane / kOct;
  size_t tok0, seq = 0;    // first token of the tile, counted over all rows; its long group
  int nt, wtile = 0;       // tokens of the tile; its index in the long group
  if constexpr (kWhole) {
    // block = seq * tiles_launch + tile; the quotient by the host's fl(2^32 / tiles_launch) + 1 where
    // that is exact (a division by a run-time value costs dozens of instructions ahead of the loads)
    const unsigned wseq = a.tiles_launch == 1 ? block
                        : a.launch_magic ? __umulhi(block, a.launch_magic)
                                         : block / (unsigned)a.tiles_launch;
    wtile = a.tile_first + (int)(block - wseq * (unsigned)a.tiles_launch);
    seq = wseq;
    tok0 = seq * (size_t)a.seq_tokens + (wtile ? a.first_tokens + (size_t)(wtile - 1) * kTile : 0);
    nt = wtile ? kTile : a.first_tokens;
  } else {
    tok0 = (size_t)block * a.tile_stride;
    const size_t left = a.n_tokens - tok0;
    nt = !SHORT ? kTile : left < (size_t)a.tile_stride ? (int)left : a.tile_stride;
  }
  const v8h* src = reinterpret_cast<const v8h*>(a.x) + tok0 * kOct + c8;

  v8h x[kLoads];                                          // token 32w + kSlots i + ts, read exactly once
  if (!SHORT || nt == kTile) {
    const v8h* p = src + (size_t)(32 * wave + ts) * kOct;
#pragma unroll
    for (int i = 0; i < kLoads; ++i) x[i] = __builtin_nontemporal_load(p + (size_t)i * kSlots * kOct);
  } else {
#pragma unroll
    for (int i = 0; i < kLoads; ++i)
      x[i] = __builtin_nontemporal_load(src + (size_t)min(32 * wave + kSlots * i + ts, nt - 1) * kOct);
  }

  if constexpr (kWhole) {
    // ---- 1 + 2. the group's extrema from the partials of the first pass; parameters and thresholds
    if (tid < D) {
      const int c = tid;
      const _Float16* part = seq_partials<D, BITS>(a, seq);
      _Float16 lo = part[c], hi = part[D + c];
      for (int sp0 = 1; sp0 < a.splits; sp0 += 8) {          // eight partials in flight (repeated past the end)
        _Float16 l[8], h[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int sp = min(sp0 + i, a.splits - 1);
          l[i] = part[(sp * 2 + 0) * D + c];
          h[i] = part[(sp * 2 + 1) * D + c];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          lo = (_Float16)fminf((float)lo, (float)l[i]);
          hi = (_Float16)fmaxf((float)hi, (float)h[i]);
        }
      }
      const uint16_t mbits = canonical_zero(__builtin_bit_cast(uint16_t, lo));
      const double alpha = h_to_double(mbits);
      const double range = ((double)(float)hi - alpha) + 0.0;
      if (wtile == a.tiles_seq - 1) {          // one block per group stores the parameters
        a.scale[seq * D + c] = (float)(range / (double)L);
        a.minv[seq * D + c] = mbits;
      }
      if constexpr (kWide) {
        s_alpha[c] = __builtin_bit_cast(_Float16, mbits);
        s_rinv[c] = range > 0.0 ? (double)L / range : 0.0;
      } else {
#pragma unroll
        for (int k = 1; k <= L; ++k)
          s_thr[(k - 1) * D + c] = __builtin_bit_cast(_Float16, threshold_bits(alpha, range, k, L));
      }
    }
    __syncthreads();   // in the group's last tile this also orders the reads above before the
                       // block's own code words, which replace the partials
  } else if constexpr (AXIS == CQ_AXIS_CHANNEL) {
    // ---- 1. per-channel extrema over the wave's 32 tokens
    v8h mn = x[0], mx = x[0];
#pragma unroll
    for (int i = 1; i < kLoads; ++i) {
      mn = __builtin_elementwise_min(mn, x[i]);
      mx = __builtin_elementwise_max(mx, x[i]);
    }
    store_extrema<kOct>(mn, mx, lane, s_part[0][wave], s_part[1][wave]);
    __syncthreads();
    // ---- 2. one thread per (group, channel), two where there are three thresholds: stored parameters and thresholds
    constexpr int kWavesPerGroup = GROUP / 32;
    for (int at = tid; at < kParts * NG * D; at += kThreads) {
      const int part = at / (NG * D), item = at % (NG * D), g = item / D, c = item % D;
      _Float16 lo = s_part[0][g * kWavesPerGroup][c], hi = s_part[1][g * kWavesPerGroup][c];
#pragma unroll
      for (int w = 1; w < kWavesPerGroup; ++w) {
        lo = (_Float16)fminf((float)lo, (float)s_part[0][g * kWavesPerGroup + w][c]);
        hi = (_Float16)fmaxf((float)hi, (float)s_part[1][g * kWavesPerGroup + w][c]);
      }
      const uint16_t mbits = canonical_zero(__builtin_bit_cast(uint16_t, lo));
      const double alpha = h_to_double(mbits);
      const double range = ((double)(float)hi - alpha) + 0.0;
      if (part == 0 && g * GROUP < nt) {       // a short last tile holds whole groups only
        const size_t meta = ((size_t)block * NG + g) * D + c;
        a.scale[meta] = (float)(range / (double)L);
        a.minv[meta] = mbits;
      }
      if constexpr (kWide) {
        s_alpha[g * D + c] = __builtin_bit_cast(_Float16, mbits);
        s_rinv[g * D + c] = range > 0.0 ? (double)L / range : 0.0;
      } else {
#pragma unroll
        for (int k = 1; k <= L; ++k)
          if (kParts == 1 || (k > 1) == (part == 1))
            s_thr[(g * L + (k - 1)) * D + c] =
                __builtin_bit_cast(_Float16, threshold_bits(alpha, range, k, L));
      }
    }
    __syncthreads();
  }
  if constexpr (AXIS == CQ_AXIS_CHANNEL) {
    // ---- 3. codes
    const int g = (32 * wave) / kG;
    if constexpr (kWide) {
      double al[8], ri[8];
      float al32[8], ri32[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        al32[j] = (float)s_alpha[g * D + c8 * 8 + j];
        al[j] = (double)al32[j];
        ri[j] = s_rinv[g * D + c8 * 8 + j];
        ri32[j] = (float)ri[j];
      }
#pragma unroll
      for (int i = 0; i < kLoads; ++i) {
        const int tok = 32 * wave + kSlots * i + ts;
        uint32_t w0, w1;
        octet_words<BITS>(x[i], al, ri, al32, ri32, w0, w1);
        if constexpr (BITS == 4) {
          s_codes[tok * kWords + c8] = w0;
        } else {
          s_codes[tok * kWords + 2 * c8] = w0;
          s_codes[tok * kWords + 2 * c8 + 1] = w1;
        }
      }
    } else {
    v8h thr[L];
#pragma unroll
    for (int k = 0; k < L; ++k) thr[k] = *reinterpret_cast<const v8h*>(&s_thr[(g * L + k) * D + c8 * 8]);
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      uint32_t bits = octet_codes<BITS>(x[i], thr);
      const int tok = 32 * wave + kSlots * i + ts;
      if constexpr (BITS == 1) {
        bits <<= 24 - 8 * (c8 & 3);
        bits |= other_lane<0xB1>(bits);
        bits |= other_lane<0x4E>(bits);
        if ((c8 & 3) == 0) s_codes[tok * kWords + (c8 >> 2)] = bits;
      } else {
        bits <<= 16 - 16 * (c8 & 1);
        bits |= other_lane<0xB1>(bits);
        if ((c8 & 1) == 0) s_codes[tok * kWords + (c8 >> 1)] = bits;
      }
    }
    }
  } else {
    // ---- 1. per-token extrema over the lanes of a channel group
    constexpr int kLanesPerGroup = GROUP / 8;
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const v8h xi = x[i];
      const v4h qa = __builtin_shufflevector(xi, xi, 0, 1, 2, 3);
      const v4h qb = __builtin_shufflevector(xi, xi, 4, 5, 6, 7);
      const v4h lo4 = __builtin_elementwise_min(qa, qb), hi4 = __builtin_elementwise_max(qa, qb);
      const v2h lo = __builtin_elementwise_min(__builtin_shufflevector(lo4, lo4, 0, 1),
                                               __builtin_shufflevector(lo4, lo4, 2, 3));
      const v2h hi = __builtin_elementwise_max(__builtin_shufflevector(hi4, hi4, 0, 1),
                                               __builtin_shufflevector(hi4, hi4, 2, 3));
      v2h st = {(_Float16)fminf((float)lo[0], (float)lo[1]),
                (_Float16)(-fmaxf((float)hi[0], (float)hi[1]))};                    // {min, -max}
      // over 4 to 32 lanes, in the vector unit as far as a row of 16 reaches (each step finds equal values in the
      // lanes that the ones before it have joined, so a mirror does for a distance of 4 or 8)
      auto join = [&](uint32_t other) { st = __builtin_elementwise_min(st, __builtin_bit_cast(v2h, other)); };
      join(other_lane<0xB1>(__builtin_bit_cast(uint32_t, st)));
      join(other_lane<0x4E>(__builtin_bit_cast(uint32_t, st)));
      if constexpr (kLanesPerGroup >= 8) join(other_lane<0x141>(__builtin_bit_cast(uint32_t, st)));
      if constexpr (kLanesPerGroup >= 16) join(other_lane<0x140>(__builtin_bit_cast(uint32_t, st)));
      if constexpr (kLanesPerGroup >= 32) join(__shfl_xor(__builtin_bit_cast(uint32_t, st), 16));
      if ((c8 % kLanesPerGroup) == 0) {
        const int tok = 32 * wave + kSlots * i + ts;
        s_stat[tok * kPerTok + c8 / kLanesPerGroup][0] = st[0];
        s_stat[tok * kPerTok + c8 / kLanesPerGroup][1] = -st[1];
      }
    }
    __syncthreads();
    // ---- 2. one thread per (token, channel group), or two
    for (int both = tid; both < kParts * kTile * NG; both += kThreads) {
      const int part = both / (kTile * NG), item = both % (kTile * NG);
      const int at = item / NG * kPerTok + item % NG;
      const uint16_t mbits = canonical_zero(__builtin_bit_cast(uint16_t, s_stat[at][0]));
      const double alpha = h_to_double(mbits);
      const double range = ((double)(float)s_stat[at][1] - alpha) + 0.0;
      if (part == 0 && item < nt * NG) {
        const size_t meta = tok0 * NG + item;
        a.scale[meta] = (float)(range / (double)L);
        a.minv[meta] = mbits;
      }
      if constexpr (kWide) {
        s_alpha[at] = __builtin_bit_cast(_Float16, mbits);
        s_rinv[at] = range > 0.0 ? (double)L / range : 0.0;
      } else {
#pragma unroll
        for (int k = 1; k <= L; ++k)
          if (kParts == 1 || (k > 1) == (part == 1)) s_thr[at * 4 + (k - 1)] = __builtin_bit_cast(_Float16, threshold_bits(alpha, range, k, L));
      }
    }
    __syncthreads();
    // ---- 3. codes
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const int tok = 32 * wave + kSlots * i + ts, item = tok * kPerTok + c8 / kLanesPerGroup;
      if constexpr (kWide) {
        const float a32 = (float)s_alpha[item];
        const double a1 = (double)a32, r1 = s_rinv[item];
        const float r32 = (float)r1;
        const double al[8] = {a1, a1, a1, a1, a1, a1, a1, a1}, ri[8] = {r1, r1, r1, r1, r1, r1, r1, r1};
        const float al32[8] = {a32, a32, a32, a32, a32, a32, a32, a32};
        const float ri32[8] = {r32, r32, r32, r32, r32, r32, r32, r32};
        uint32_t w0, w1;
        octet_words<BITS>(x[i], al, ri, al32, ri32, w0, w1);
        if constexpr (BITS == 4) {
          s_codes[tok * kWords + c8] = w0;
        } else {
          s_codes[tok * kWords + 2 * c8] = w0;
          s_codes[tok * kWords + 2 * c8 + 1] = w1;
        }
        continue;
      }
      v8h thr[L];
#pragma unroll
      for (int k = 0; k < L; ++k) {
        const _Float16 t = s_thr[item * 4 + k];
        thr[k] = (v8h){t, t, t, t, t, t, t, t};
      }
      uint32_t bits = octet_codes<BITS>(x[i], thr);
      if constexpr (BITS == 1) {
        bits <<= 24 - 8 * (c8 & 3);
        bits |= other_lane<0xB1>(bits);
        bits |= other_lane<0x4E>(bits);
        if ((c8 & 3) == 0) s_codes[tok * kWords + (c8 >> 2)] = bits;
      } else {
        bits <<= 16 - 16 * (c8 & 1);
        bits |= other_lane<0xB1>(bits);
        if ((c8 & 1) == 0) s_codes[tok * kWords + (c8 >> 1)] = bits;
      }
    }
  }
  __syncthreads();
  // ---- the tile's words are contiguous in memory: 16 bytes per thread (8 where a token has 8 bytes
  // of codes, as a group may then start between two 16-byte boundaries)
  if constexpr (kWords >= 4) {
    v4u* dst = reinterpret_cast<v4u*>(a.codes + tok0 * kWords);
    for (int i = tid; i < nt * (kWords / 4); i += kThreads)
      dst[i] = *reinterpret_cast<const v4u*>(&s_codes[i * 4]);
  } else {
    v2u* dst = reinterpret_cast<v2u*>(a.codes + tok0 * kWords);
    for (int i = tid; i < nt; i += kThreads) dst[i] = *reinterpret_cast<const v2u*>(&s_codes[i * 2]);
  }
}

// (one- and two-bit codes of up to 128 channels: eight waves per SIMD, which the compiler otherwise
// misses by two registers for some groups)
template <int D, int AXIS, int BITS, int GROUP, bool SHORT = true>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(D <= 128 && BITS <= 2 ? 8 : 1)))
quantize_tile_kernel(const QArgs a) {
  __shared__ TileMem<D, AXIS, BITS, GROUP> sm;
  // An XCD (every eighth block) takes eight tiles in a row, a quarter of a megabyte at 128 channels, not every eighth tile:
  // us, keys and values, every eighth / eight in a row: 1024 rows x 16384 tokens, 1 bit 1764 / 1669, 2 bits 1838 / 1809, 512 x
  // 8192, 1 bit 389 / 389, 4 bits 480 / 475.  (Runs of 2: 1760; 4: 1687; 64: 1687; 256: 1663, but 2 bits in groups of 32 only as fast as
  // without; 4096: slower there.)  Not with 8 bits, which lose: 256 x 16384 552 / 562.  Not with 64 channels, half the bytes
  // to a run: one tensor, 1 bit, loses 3 to 7 % below 64 MB (256 x 4096 23.4 / 24.5) and gains nothing above, 2 and 4 bits
  // are the same.  Not for long groups, the same within 1.5 %.  (The pair kernel below keeps every eighth tile: with 128
  // channels the same within 2 %, but for 64 x 3328, 4 bits, 3 % less; with 256 channels runs take 1 to 5 % less; with 64 up to
  // 8 % more.)
  unsigned block = blockIdx.x;
  if constexpr (GROUP != 0 && D > 64 && BITS != 8) {
    const unsigned base = block & ~63u;
    if (base + 64 <= gridDim.x) block = base + ((block & 7) << 3) + ((block >> 3) & 7);
  }
  quantize_tile<D, AXIS, BITS, GROUP, SHORT>(a, block, sm);
}

// Keys and values in one launch, the first n_first blocks on the keys (channel-wise, KGROUP).
template <int D, int BITS, int KGROUP, int VAXIS, int VGROUP>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(D <= 128 && BITS <= 2 ? 8 : 1)))
quantize_pair_kernel(const QArgs keys, const QArgs values, unsigned n_first) {
  __shared__ union {
    TileMem<D, CQ_AXIS_CHANNEL, BITS, KGROUP> k;
    TileMem<D, VAXIS, BITS, VGROUP> v;
  } sm;
  if constexpr (VAXIS == CQ_AXIS_CHANNEL && VGROUP == KGROUP) {
    const QArgs a = blockIdx.x < n_first ? keys : values;
    quantize_tile<D, CQ_AXIS_CHANNEL, BITS, KGROUP>(a, blockIdx.x < n_first ? blockIdx.x : blockIdx.x - n_first, sm.k);
  } else {
    if (blockIdx.x < n_first) quantize_tile<D, CQ_AXIS_CHANNEL, BITS, KGROUP>(keys, blockIdx.x, sm.k);
    else quantize_tile<D, VAXIS, BITS, VGROUP>(values, blockIdx.x - n_first, sm.v);
  }
}

// One tensor as the launches below see it.
struct Task {
  QArgs a{};
  int axis = 0, kernel_group = 0;        // GROUP of the kernel: 0 = long groups
  size_t blocks = 0, n_seq = 0;          // tile blocks; long groups
};

// n_vis is a multiple of a channel-wise group.
inline Task make_task(const void* x_f16, const cq_qtensor_t& out, size_t n_tokens, int bits, int axis, int group) {
  Task t;
  t.axis = axis;
  t.a.x = static_cast<const __half*>(x_f16);
  t.a.codes = out.codes; t.a.scale = out.scale; t.a.minv = out.min;
  t.a.n_tokens = n_tokens;
  t.a.tile_stride = kTile;
  const bool flat = axis == CQ_AXIS_TOKEN || group == 32 || group == 64 || group == 128;
  t.kernel_group = flat ? group : kTile;
  if (!flat && group > kTile) {
    t.kernel_group = 0;
    t.n_seq = n_tokens / group;
    t.a.seq_tokens = group;
    t.a.tiles_seq = ceil_div(group, kTile);
    t.a.first_tokens = group - (t.a.tiles_seq - 1) * kTile;
    // enough blocks in the first pass to fill the chip, as far as the last tile's code words hold
    // their partials
    const size_t want = (2048 + t.n_seq - 1) / t.n_seq;
    t.a.splits = want < 4 ? 4 : want < (size_t)max_splits(bits) ? (int)want : max_splits(bits);
    t.blocks = t.n_seq * (size_t)t.a.tiles_seq;
    return t;
  }
  if (!flat) t.a.tile_stride = group;          // a short group is a tile of its own
  t.blocks = (n_tokens + t.a.tile_stride - 1) / t.a.tile_stride;
  return t;
}

// Whether the launches of a tensor stay within 2^32 - 1 threads, which HIP takes.
inline bool launchable(const Task& t) {
  const size_t most = 0xffffffffu / kThreads;
  return t.blocks <= most && t.n_seq * (size_t)t.a.splits <= most;
}

// long groups: extrema pass, all tiles but the last of every group, the last tiles; u: NULL, or a second
// tensor with long groups
template <int D, int BITS>
hipError_t launch_long_groups(const Task& t, const Task* u, hipStream_t stream) {
  QArgs a = t.a, b = u ? u->a : t.a;
  const size_t na = t.n_seq, nb = u ? u->n_seq : 0;
  row_extrema_kernel<D, BITS><<<dim3((unsigned)(na * a.splits + nb * b.splits)), dim3(kThreads), 0, stream>>>(
      a, b, (unsigned)(na * a.splits));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  auto share = [](QArgs& q, size_t n_seq, int first, int count) -> unsigned {
    q.tile_first = first;
    q.tiles_launch = count;
    const unsigned long long blocks = (unsigned long long)n_seq * (unsigned)count;
    q.launch_magic = count > 1 && blocks * (unsigned)count < (1ull << 32)
                         ? (unsigned)((1ull << 32) / (unsigned)count + 1) : 0u;
    return (unsigned)blocks;
  };
  for (int last = 0; last < 2; ++last) {
    const unsigned ba = last ? share(a, na, a.tiles_seq - 1, 1) : share(a, na, 0, a.tiles_seq - 1);
    if (u) {
      const unsigned bb = last ? share(b, nb, b.tiles_seq - 1, 1) : share(b, nb, 0, b.tiles_seq - 1);
      quantize_pair_kernel<D, BITS, 0, CQ_AXIS_CHANNEL, 0><<<dim3(ba + bb), dim3(kThreads), 0, stream>>>(a, b, ba);
    } else {
      quantize_tile_kernel<D, CQ_AXIS_CHANNEL, BITS, 0><<<dim3(ba), dim3(kThreads), 0, stream>>>(a);
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int D, int BITS>
hipError_t launch_tiles(const Task& t, hipStream_t stream) {
  if (t.kernel_group == 0) return launch_long_groups<D, BITS>(t, nullptr, stream);
  void (*kern)(const QArgs) = nullptr;
  const int g = t.kernel_group;
  if (t.axis == CQ_AXIS_CHANNEL)               // 128: also one group per short tile
    kern = g == 32 ? quantize_tile_kernel<D, CQ_AXIS_CHANNEL, BITS, 32>
         : g == 64 ? quantize_tile_kernel<D, CQ_AXIS_CHANNEL, BITS, 64> : quantize_tile_kernel<D, CQ_AXIS_CHANNEL, BITS, 128>;
  else if (g == 32) kern = quantize_tile_kernel<D, CQ_AXIS_TOKEN, BITS, 32>;
  else if (g == 64) kern = quantize_tile_kernel<D, CQ_AXIS_TOKEN, BITS, 64>;
  if constexpr (D >= 128) { if (t.axis == CQ_AXIS_TOKEN && g == 128) kern = quantize_tile_kernel<D, CQ_AXIS_TOKEN, BITS, 128>; }
  if constexpr (D >= 256) { if (t.axis == CQ_AXIS_TOKEN && g == 256) kern = quantize_tile_kernel<D, CQ_AXIS_TOKEN, BITS, 256>; }
  // Token-wise two-bit codes are the one kernel that the path for short tiles slows down (456 rows x
  // 2688 tokens x 128 channels: 67.2 us without it, 69.5 with it; the others differ by less than 1 %).
  if constexpr (D == 128 && BITS == 2) {
    if (t.axis == CQ_AXIS_TOKEN && t.a.n_tokens % kTile == 0)
      kern = g == 32 ? quantize_tile_kernel<D, CQ_AXIS_TOKEN, BITS, 32, false>
           : g == 64 ? quantize_tile_kernel<D, CQ_AXIS_TOKEN, BITS, 64, false>
                     : quantize_tile_kernel<D, CQ_AXIS_TOKEN, BITS, 128, false>;
  }
  if (!kern) return hipErrorInvalidValue;
  kern<<<dim3((unsigned)t.blocks), dim3(kThreads), 0, stream>>>(t.a);
  return hipGetLastError();
}

// The kernel that takes both tensors in one launch; NULL where there is none.  The pairs that callers
// combine: groups of tokens for the keys with values token-wise over the head or in groups of
// tokens of their own.
template <int D, int BITS>
auto pair_kernel(const Task& k, const Task& v) -> void (*)(const QArgs, const QArgs, unsigned) {
  if (k.axis != CQ_AXIS_CHANNEL) return nullptr;
  const int kg = k.kernel_group, vg = v.kernel_group;
  if (v.axis == CQ_AXIS_TOKEN) {
    if (vg != D) return nullptr;
    return kg == 32 ? quantize_pair_kernel<D, BITS, 32, CQ_AXIS_TOKEN, D>
         : kg == 64 ? quantize_pair_kernel<D, BITS, 64, CQ_AXIS_TOKEN, D>
         : kg == 128 ? quantize_pair_kernel<D, BITS, 128, CQ_AXIS_TOKEN, D> : nullptr;
  }
  if (vg == 64)
    return kg == 32 ? quantize_pair_kernel<D, BITS, 32, CQ_AXIS_CHANNEL, 64>
         : kg == 64 ? quantize_pair_kernel<D, BITS, 64, CQ_AXIS_CHANNEL, 64>
         : kg == 128 ? quantize_pair_kernel<D, BITS, 128, CQ_AXIS_CHANNEL, 64> : nullptr;
  if (vg == 128)
    return kg == 32 ? quantize_pair_kernel<D, BITS, 32, CQ_AXIS_CHANNEL, 128>
         : kg == 64 ? quantize_pair_kernel<D, BITS, 64, CQ_AXIS_CHANNEL, 128>
         : kg == 128 ? quantize_pair_kernel<D, BITS, 128, CQ_AXIS_CHANNEL, 128> : nullptr;
  return nullptr;
}

// Largest tensor (elements) whose keys and values go out together.  Two launches leave a part of the
// chip idle at the end of the first and all of it waiting at the start of the second: together,
// 1 to 8 bits, 3.4 M elements take 7-10 us instead of 12-14, 27 M (D = 128) 10-20 % less, 67 M 4-12 %
// less (between 2 % more and 8 % less at D = 256).  Beyond that the streams of both tensors only
// disturb each other: 134 M elements between 3 % less and 5 % more, 537 M up to 6 % more.
constexpr size_t kPairElements = (size_t)80 << 20;

// Up to two tensors (v: NULL for one) in as few launches as their kernels allow.
template <int D, int BITS>
hipError_t launch_tasks(const Task& k, const Task* v, hipStream_t stream) {
  if (v && k.a.n_tokens * D <= kPairElements) {
    if (k.kernel_group == 0 && v->kernel_group == 0) return launch_long_groups<D, BITS>(k, v, stream);
    if (auto kern = pair_kernel<D, BITS>(k, *v)) {
      kern<<<dim3((unsigned)(k.blocks + v->blocks)), dim3(kThreads), 0, stream>>>(k.a, v->a, (unsigned)k.blocks);
      return hipGetLastError();
    }
  }
  const hipError_t e = launch_tiles<D, BITS>(k, stream);
  return e != hipSuccess || !v ? e : launch_tiles<D, BITS>(*v, stream);
}

template <int D>
hipError_t launch_quantize_dim(const QuantizeJob* jobs, int n_jobs, size_t n_tokens, int bits, hipStream_t stream) {
  Task t[2];
  for (int i = 0; i < n_jobs; ++i) {
    t[i] = make_task(jobs[i].x_f16, jobs[i].out, n_tokens, bits, jobs[i].axis, jobs[i].group);
    if (!launchable(t[i])) return hipErrorInvalidConfiguration;
  }
  const Task* v = n_jobs > 1 ? &t[1] : nullptr;
  switch (bits) {
    case 1: return launch_tasks<D, 1>(t[0], v, stream);
    case 2: return launch_tasks<D, 2>(t[0], v, stream);
    case 4: return launch_tasks<D, 4>(t[0], v, stream);
    case 8: return launch_tasks<D, 8>(t[0], v, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace
}  // namespace cq

#endif  // CQ_QUANTIZE_TILE_H_
