// Decode attention over the packed cache for the layouts that the fused and the streaming kernels do
// not take (gfx950): head_dim 64, 128 or 256, 1-, 2-, 4- or 8-bit codes, channel-wise keys in groups
// of any number of tokens (with 128 channels the whole sequence is the fused kernel's, whatever its length), values
// token-wise with one group per token or channel-wise in groups of any number of tokens, any
// number of query heads per KV head.
//
//   logits pass   (row, head set, chunk of the visual tokens) or (row, chunk of the fp16 tail) per
//                 workgroup of 4 waves: raw logits in fp32 and the extrema of the chunk to the workspace
//   values pass   the same division of the tokens into chunks of their own: g of Sec. 3.2 from the row's
//                 extrema, weights, one partial (m, l, acc[D]) of the joint softmax per (head, chunk)
//                 the workgroup that stores the last partial of its heads merges them all
//
// Both contractions over packed codes run on the int8 matrix cores as in decode_fused.hip (codes
// picked out of a word by AND masks, the other operand as four signed base-256 digits of a 29-bit
// fixed-point number, 4 query heads = 16 matrix rows), here for any head_dim that is a multiple of 64.
// A wave works for itself: it owns whole blocks of up to 128 tokens of one key group (logits) or a
// run of 64-token tiles (values); groups and the row's end cut blocks and tiles short, a short one
// reads its last token again and the surplus is neither stored nor weighted.
//
// Precision.  Keys: one fixed-point scale per key group and head set, 30 bits, results put together in fp64.
// Values: a scale per head that follows the products weight * scale (see Scales), sums in fp32.  A
// host model of the sums, 3328 tokens, relative to fp64: 0.6e-7 to 2e-7 whether or not a token's scale stands
// out a thousandfold (fp32 multiply-adds over dequantized values: 2e-7 to 4e-7; one scale for all heads set by
// the largest token scale: 6e-7 to 1e-5); 1e-6 where a wave takes 4096 tokens of very uneven weights
// (logits with a deviation of 6; fp32 2e-7), a two hundredth of the output's rounding.  Following the
// products costs a small call 0.1 to 0.2 us.
//
// Both passes run as one launch (tile_row_kernel) where that is faster, see plan_one_launch.
//
// Bound: on small calls latency - in each wave a chain of few round trips to memory: all that a wave needs first
// is asked for at once (the query, its first codes and parameters; its first value tile, then the
// extrema), a key block's codes together, a share of the tail together.  On large ones the issue of vector instructions; 16 waves share a CU and hide each other's
// latency.  Against the shape-agnostic kernels, which dequantize element by element: 64 rows x
// 3003 tokens, 2 bits, whole-sequence keys and values 618 -> 15.6 us; 64 rows x 3328 tokens of 64
// channels, 1 bit, 422 -> 14.1 us.  Over key and value groups from 1 to 48 tokens, head_dim 64 to 256
// and 1 and 8 bits they are 1.8 (value groups of one token) to 26 times as fast, and over 230 drawn
// layouts and tails never slower, so they take every layout they can.
#include <hip/hip_fp16.h>

#include <cfloat>

#include "cq_internal.h"
#include "decode_device.h"
#include "decode_fold.h"
#include "decode_meet.h"

namespace cq {
namespace {

constexpr int kWaves = 4;
constexpr int kThreads = kWaves * 64;
constexpr int kKeyBlock = 128;       // most tokens per key block (8 tiles of 16)
constexpr int kValTile = 64;         // tokens per value tile
constexpr int kTextShare = 32;       // tokens of the fp16 tail per wave and round
constexpr int kTextBlock = kWaves * kTextShare;
// one launch: chunks are whole units of 128 tokens, so many at least and at most; workgroups to aim at
constexpr int kUnit = 128, kRowMinUnits = 4, kRowMaxUnits = 8, kRowTarget = 768;
constexpr int kRowMost = 4096, kRowMostShort = 512, kRowMostChunks = 56;      // see plan_one_launch
constexpr int kRowMostAll = 250000, kRowMostWide = 100000, kRowLeast64 = 150000;
constexpr int kMaxRun = 1024;        // value tiles between two folds of the int32 digit sums (2^20 each)

struct TileArgs {
  const __half* q;
  const uint32_t* k_codes; const float* k_scale; const uint16_t* k_min;
  const uint32_t* v_codes; const float* v_scale; const uint16_t* v_min;
  const __half* k_text; const __half* v_text;
  int g, sets, n_vis, n_text, n_text_cap;    // sets = ceil(g / 4)
  const int32_t* n_text_dev;   // NULL, or the tail length in device memory (n_text is then its bound)
  int k_group, k_bpg, k_groups;   // tokens per key group, blocks per group, groups per row
  int k_block;                    // most tokens per key block
  int v_group, v_tpg, v_groups;   // tokens per value group (token-wise: n_vis), tiles per group, groups per row
  int ca, ca_base, ca_rem;     // logits pass: chunks per row, in key blocks
  int cb, cb_base, cb_rem;     // values pass: chunks per row, in value tiles
  int ct, ct_tokens;           // chunks of the fp16 tail per row, tokens per chunk
  // logits pass on its own: logits of a second set of 16-bit keys [rows][x_tokens][D] in the same launch
  const __half* x_keys; int x_tokens, x_ct, x_ct_tokens; float* x_logits; float* x_minmax;
  float* ws_logits;            // [B*Hq][n_vis + n_text]
  float* ws_minmax;            // [B*Hq][ca + ct][2]
  float* ws_partial;           // [B*Hq][cb + ct][D + 2]
  int* ws_count;               // [rows][sets] partials stored so far; NULL: no values pass follows
  // one launch (tile_row_kernel): chunks of cb_base or cb_base + 1 units of 128 tokens
  int k_bpu, v_tpu, k_blocks, v_tiles;   // key blocks and value tiles per unit, per row
  int l_stride;                // floats between the logits of two heads in LDS
  unsigned slots_magic;        // fl(2^32 / (cb + ct)) + 1, or 0 when there is one slot
  u64* ws_words; u64* ws_tags; // [B*Hq][cb][2] words of the exchange, [rows][sets] counts under the call's tag
  u64 tag; int patience;
  __half* out;
  int calib_mode; float tau1, tau2, gamma, delta, softmax_scale;
};

// How the codes of a token become the operand registers of a lane.  A matrix product takes 64 codes,
// 16 per lane (4 registers of 4 bytes); a token of D codes fills D / 64 products.  Lane row kb holds
// `words` consecutive words of its token, register p is variant p % kV (code of every byte) of word
// p / kV.  One-bit codes of 64 channels are the exception: two words for four lane rows, so a lane
// row holds half a word, the lower or the upper half of every byte.
// Codes by the lower masks of decode_device.h.
template <int D, int BITS>
struct Operand {
  static constexpr int kProducts = D / 64;
  static constexpr int kV = 8 / BITS;                       // variants (codes per byte)
  static constexpr bool kHalf = D * BITS < 128;             // half a word per lane row
  static constexpr int kWords = kHalf ? 1 : D * BITS / 128; // words per lane
  static constexpr int kRowWords = D * BITS / 32;           // words per token
  __device__ static int first_word(int kb) { return kHalf ? kb >> 1 : kb * kWords; }
  __device__ static int shift(int kb) { return kHalf ? 4 * (kb & 1) : 0; }
  // channel of operand byte y of register p in lane row kb
  __device__ static int channel(int kb, int p, int y) {
    const int e = kHalf ? 0 : p / kV, v = kHalf ? p + 4 * (kb & 1) : p % kV;
    return (32 / BITS) * (first_word(kb) + e) + code_in_word<BITS>(y, v);
  }
  // 1 / (what a code of 1 is worth in register p)
  __device__ static float weight(int p) {
    return low_weight<BITS>(p % kV);
  }
  __device__ static int reg(const uint32_t (&w)[kWords], int p, int sh) {
    return kHalf ? operand_low<BITS>(w[0] >> sh, p) : operand_low<BITS>(w[p / kV], p % kV);
  }
};

template <int N>
__device__ inline void load_words(uint32_t (&w)[N], const uint32_t* p) {
  if constexpr (N == 1) {
    w[0] = *p;
  } else if constexpr (N == 2) {
    const v2i t = *reinterpret_cast<const v2i*>(p);
    w[0] = (uint32_t)t[0];
    w[1] = (uint32_t)t[1];
  } else {
#pragma unroll
    for (int e = 0; e < N / 4; ++e) {
      const v4i t = reinterpret_cast<const v4i*>(p)[e];
#pragma unroll
      for (int u = 0; u < 4; ++u) w[4 * e + u] = (uint32_t)t[u];
    }
  }
}

// k / per without a division where there is nothing to divide: one part, or parts of one (a division
// by a value that is only known at run time takes about 40 instructions)
__device__ inline int part_of(int k, int per) { return per == 1 ? k : k < per ? 0 : k / per; }

// min and max of the workgroup's waves for the 16 heads of a text workgroup or the 4 of a head set:
// lane h of wave 0 stores head h
__device__ inline void store_extrema(float (*red)[16][2], int n_heads, float* mm, size_t pitch) {
  __syncthreads();
  const int h = threadIdx.x;
  if (h < n_heads) {
    float lo = FLT_MAX, hi = -FLT_MAX;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      lo = fminf(lo, red[w][h][0]);
      hi = fmaxf(hi, red[w][h][1]);
    }
    mm[h * pitch] = lo;
    mm[h * pitch + 1] = hi;
  }
}

// ===================================================================================== logits pass
// A workgroup's share of the fp16 tail: all query heads of the KV head, 16 at a time, on the fp16
// matrix cores (products of fp16 numbers are exact in fp32).  keys: the row's first text key.
struct TextSpan {
  const __half* keys;          // the row's first key
  int n, chunk_tokens;
  float* logits;               // of the row's first head and first token
  size_t pitch;                // between two heads
  float* minmax;               // of the row's first head and the chunk
  size_t mm_pitch;
};
template <int D>
__device__ inline void text_logits(const TileArgs& a, const TextSpan& x, size_t row, int chunk, float (*red)[16][2]) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n16 = lane & 15, kb = lane >> 4;
  const int t0 = chunk * x.chunk_tokens, t1 = min(t0 + x.chunk_tokens, x.n);
  for (int h0 = 0; h0 < a.g; h0 += 16) {
    const int nh = min(16, a.g - h0);
    const size_t head0 = row * a.g + h0;
    v8h A[D / 32];
#pragma unroll
    for (int s = 0; s < D / 32; ++s) {
      const v8h z = {0, 0, 0, 0, 0, 0, 0, 0};
      A[s] = n16 < nh ? *reinterpret_cast<const v8h*>(a.q + (head0 + n16) * D + 32 * s + 8 * kb) : z;
    }
    float mn[4], mx[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) { mn[r] = FLT_MAX; mx[r] = -FLT_MAX; }
    // a round's tiles of a wave in flight together: a tail's workgroup is short, and waits once
    constexpr int kFly = kTextShare / 16;
    for (int tb = t0 + 16 * wave; tb < t1; tb += 16 * kWaves * kFly) {
      v8h kv[kFly][D / 32];
#pragma unroll
      for (int u = 0; u < kFly; ++u) {
        const __half* kp = x.keys + (size_t)min(tb + 16 * kWaves * u + n16, t1 - 1) * D + 8 * kb;
#pragma unroll
        for (int s = 0; s < D / 32; ++s) kv[u][s] = *reinterpret_cast<const v8h*>(kp + 32 * s);
      }
#pragma unroll
      for (int u = 0; u < kFly; ++u) {
        const int tok = tb + 16 * kWaves * u + n16;
        v4f c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < D / 32; ++s) c = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[s], kv[u][s], c, 0, 0, 0);
        if (tok < t1) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {        // result rows 4 kb + r are heads
            if (4 * kb + r < nh) {
              const float s = c[r] * a.softmax_scale;
              x.logits[(h0 + 4 * kb + r) * x.pitch + tok] = s;
              mn[r] = fminf(mn[r], s);
              mx[r] = fmaxf(mx[r], s);
            }
          }
        }
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float lo = row_min(mn[r]), hi = row_max(mx[r]);
      if (n16 == 0) {
        red[wave][4 * kb + r][0] = lo;
        red[wave][4 * kb + r][1] = hi;
      }
    }
    store_extrema(red, nh, x.minmax + h0 * x.mm_pitch, x.mm_pitch);
    __syncthreads();
  }
}

// The wave's share of the key blocks b0 .. b1 of a row: logits of the set's heads, if store, to out (of head kb)
// from token tok_base on, and their extrema (of head kb).  xb: NP * 1024 bytes of LDS of the wave's own.
template <int D, int BITS>
__device__ inline void visual_logits(const TileArgs& a, size_t row, int set, int b0, int b1, int lane, int wave,
                                     uint8_t* xb, bool store, float* out, int tok_base, float& mn, float& mx) {
  using Op = Operand<D, BITS>;
  constexpr int NP = Op::kProducts;
  // tiles of 16 tokens whose codes are asked for together: a block's, as far as registers go
  constexpr int kFly = Op::kWords <= 4 ? 8 : Op::kWords == 8 ? 4 : 2;
  const int n16 = lane & 15, kb = lane >> 4;
  const int gh = min(kHeads, a.g - set * kHeads);              // live heads of the set
  const size_t head0 = row * a.g + (size_t)set * kHeads;

  // Writer of the query operand: lane l writes row l of every product (lane row l / 16, register
  // (l / 4) % 4, byte l % 4), one channel each; together the lanes cover every channel once.
  int ch[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) ch[i] = Op::channel(kb, 4 * i + ((lane >> 2) & 3), lane & 3);
  const uint8_t* x_rd = xb + (kb * 16 + (n16 >> 1)) * 16 + (n16 & 1) * 8;
  const uint32_t* kc = a.k_codes + row * (size_t)a.n_vis * Op::kRowWords + Op::first_word(kb);
  const int sh = Op::shift(kb);
  const size_t meta0 = row * (size_t)a.k_groups * D;
  const bool live = store && kb < gh;                 // result lane: head kb, token n16

  v4i A[NP];
  double bias = 0.0, inv_f = 0.0, inv_f16 = 0.0;
  int have = -1;                                               // key group of the operand in A
  int grp, t0, t1;                                             // of the block whose loads are in flight
  uint32_t w[kFly][Op::kWords];
  float s[NP];
  uint16_t m[NP];
  auto load_tiles = [&](int t) {                               // the kFly tiles from token t of the block
#pragma unroll
    for (int u = 0; u < kFly; ++u)
      load_words<Op::kWords>(w[u], kc + (size_t)min(t + 16 * u + n16, t1 - 1) * Op::kRowWords);
  };
  auto load_block = [&](int blk, int group_loaded) {           // codes, and parameters if they change
    grp = part_of(blk, a.k_bpg);
    t0 = grp * a.k_group + (blk - grp * a.k_bpg) * a.k_block;
    t1 = min(t0 + a.k_block, (grp + 1) * a.k_group);
    load_tiles(t0);
    if (grp != group_loaded) {
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        s[i] = a.k_scale[meta0 + (size_t)grp * D + ch[i]];
        m[i] = a.k_min[meta0 + (size_t)grp * D + ch[i]];
      }
    }
  };
  // the query and the first block are asked for together, so that a wave waits for memory once
  uint16_t q_raw[NP][kHeads];
#pragma unroll
  for (int i = 0; i < NP; ++i)
#pragma unroll
    for (int h = 0; h < kHeads; ++h)
      q_raw[i][h] = *reinterpret_cast<const uint16_t*>(a.q + (head0 + min(h, gh - 1)) * D + ch[i]);
  if (b0 + wave < b1) load_block(b0 + wave, -1);
  pin_order();
  float inv_w[NP], qv[NP][kHeads];
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const float wgt = Op::weight(4 * i + ((lane >> 2) & 3));
    inv_w[i] = 1.f / wgt;                                      // exact: powers of two
#pragma unroll
    for (int h = 0; h < kHeads; ++h)
      qv[i][h] = h < gh ? __half2float(__ushort_as_half(q_raw[i][h])) * wgt : 0.f;      // exact
  }
  for (int blk = b0 + wave; blk < b1; blk += kWaves) {
    if (blk != b0 + wave) load_block(blk, have);
    if (grp != have) {                                         // wave-uniform
      have = grp;
      float most = 0.f;
#pragma unroll
      for (int i = 0; i < NP; ++i) {
#pragma unroll
        for (int h = 0; h < kHeads; ++h) most = fmaxf(most, fabsf(qv[i][h] * s[i]));
      }
      // the largest operand is below 2^30: the top digit of four stays below 64
      const int F = 1 + fixed_point_shift(wave_max_nonneg(most));
      double part[kHeads] = {0.0, 0.0, 0.0, 0.0};
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const double sf = ldexp((double)s[i], F);
        v4i x;
#pragma unroll
        for (int h = 0; h < kHeads; ++h) x[h] = rounded_digits(qv[i][h], sf);
        *reinterpret_cast<v4i*>(xb + i * 1024 + lane * 16) = x;
        // 8-bit operand bytes are code - 128: the 128 comes back with the minimum
        const double f = ((double)__half2float(__ushort_as_half(m[i])) + (BITS == 8 ? 128.0 * (double)s[i] : 0.0)) * (double)inv_w[i];
#pragma unroll
        for (int h = 0; h < kHeads; ++h) part[h] = fma((double)qv[i][h], f, part[h]);
      }
      lds_publish();
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const v2i lo = lds_read_tr8(x_rd + i * 1024), hi = lds_read_tr8(x_rd + i * 1024 + 128);
        A[i] = (v4i){lo[0], lo[1], hi[0], hi[1]};
      }
      bias = head_sums(part, lane) * (double)a.softmax_scale;
      inv_f = ldexp((double)a.softmax_scale, -F);
      inv_f16 = ldexp((double)a.softmax_scale, 16 - F);
      __builtin_amdgcn_wave_barrier();
    }
    for (int t = t0; t < t1; t += 16 * kFly) {
      if (t != t0) load_tiles(t);
#pragma unroll
      for (int u0 = 0; u0 < kFly; u0 += 2) {                   // two tiles at a time
        if (t + 16 * u0 >= t1) break;                          // wave-uniform
        v4i c[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
#pragma unroll
        for (int i = 0; i < NP; ++i) {
          v4i B[2];
#pragma unroll
          for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) B[u][v] = Op::reg(w[u0 + u], 4 * i + v, sh);
#pragma unroll
          for (int u = 0; u < 2; ++u) c[u] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A[i], B[u], c[u], 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int lo = c[u][0] + (c[u][1] << 8), hi = c[u][2] + (c[u][3] << 8);
          const float s = (float)fma((double)hi, inv_f16, fma((double)lo, inv_f, bias));
          const int tok = t + 16 * (u0 + u) + n16;
          if (tok < t1) {
            if (live) out[tok - tok_base] = s;
            mn = fminf(mn, s);
            mx = fmaxf(mx, s);
          }
        }
      }
    }
  }
}

// grid: x = row, y = chunk of the tail, of the visual tokens, of the second set of keys, z = head set
// (the workgroups of 16-bit keys take all heads and leave the others of their column at once)
template <int D, int BITS>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(D == 256 ? 2 : 4)))
tile_logits_kernel(const TileArgs a) {
  __shared__ __align__(16) uint8_t s_x[kWaves][Operand<D, BITS>::kProducts * 1024];     // query operand of a wave's key group
  __shared__ float red[kWaves][16][2];
  const size_t row = blockIdx.x;
  if (blockIdx.y == 0 && blockIdx.z == 0 && a.ws_count)          // for the values pass behind this one
    for (int i = threadIdx.x; i < a.sets; i += kThreads) a.ws_count[row * a.sets + i] = 0;
  const bool tail = (int)blockIdx.y < a.ct;
  if (tail || (int)blockIdx.y >= a.ct + a.ca) {
    if (blockIdx.z != 0) return;
    const int chunk = (int)blockIdx.y - (tail ? 0 : a.ct + a.ca);
    const size_t head0 = row * a.g, pitch = (size_t)a.n_vis + a.n_text;
    TextSpan x;
    if (tail) {
      const size_t mm_pitch = (size_t)(a.ca + a.ct) * 2;
      x = {a.k_text + row * (size_t)a.n_text_cap * D, a.n_text_dev ? min(max(*a.n_text_dev, 0), a.n_text) : a.n_text,
           a.ct_tokens, a.ws_logits + head0 * pitch + a.n_vis, pitch,
           a.ws_minmax + head0 * mm_pitch + (size_t)(a.ca + chunk) * 2, mm_pitch};
    } else {
      const size_t mm_pitch = (size_t)a.x_ct * 2;
      x = {a.x_keys + row * (size_t)a.x_tokens * D, a.x_tokens, a.x_ct_tokens,
           a.x_logits + head0 * a.x_tokens, (size_t)a.x_tokens, a.x_minmax + head0 * mm_pitch + (size_t)chunk * 2,
           mm_pitch};
    }
    text_logits<D>(a, x, row, chunk, red);
    return;
  }
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n16 = lane & 15, kb = lane >> 4;
  const int set = (int)blockIdx.z, chunk = (int)blockIdx.y - a.ct;
  const int b0 = chunk_first(a.ca_base, a.ca_rem, chunk), b1 = chunk_first(a.ca_base, a.ca_rem, chunk + 1);
  const int gh = min(kHeads, a.g - set * kHeads);
  const size_t head0 = row * a.g + (size_t)set * kHeads;
  float mn = FLT_MAX, mx = -FLT_MAX;
  visual_logits<D, BITS>(a, row, set, b0, b1, lane, wave, s_x[wave], true,
                         a.ws_logits + (head0 + min(kb, gh - 1)) * ((size_t)a.n_vis + a.n_text), 0, mn, mx);
  mn = row_min(mn);
  mx = row_max(mx);
  if (n16 == 0) {
    red[wave][kb][0] = mn;
    red[wave][kb][1] = mx;
  }
  const size_t pitch = (size_t)(a.ca + a.ct) * 2;
  store_extrema(red, gh, a.ws_minmax + head0 * pitch + (size_t)chunk * 2, pitch);
}

// ===================================================================================== values pass
// The end of a workgroup of the values pass: its waves' sums become one partial (m, l, acc[D]) of the
// joint softmax per head of the set.  The workgroup that finds all other partials of its (row, head
// set) stored merges them into the output: nobody waits for anybody, and the result does not
// depend on who comes last.  Each wave's stores have reached memory (vmcnt 0) before the barrier
// that precedes the workgroup's count.  With a launch of the shared combine kernel in its place
// the two calls measured at the top of this file took 16.6 and 16.0 us.
template <int D, bool ROW>
__device__ inline void finish_chunk(const TileArgs& a, size_t row, int set, size_t head0, int gh, int slot, u64 seen,
                                    const float* m_ref, const float (*s_part)[kHeads][D],
                                    const float (*s_lm)[kHeads][2]) {
  __shared__ int s_last;
  constexpr int kPairs = D / 2;                // two channels per thread
  const int n_slots = a.cb + a.ct;
  __syncthreads();
  for (int e = threadIdx.x; e < gh * kPairs; e += kThreads) {
    const int h = e / kPairs, c = 2 * (e % kPairs);
    v2f num = {0.f, 0.f};
    float den = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      num += *reinterpret_cast<const v2f*>(&s_part[w][h][c]) + s_lm[w][h][1];
      den += s_lm[w][h][0];
    }
    if (n_slots == 1) {
      *reinterpret_cast<__half2*>(a.out + (head0 + h) * D + c) = __floats2half2_rn(num[0] / den, num[1] / den);
      continue;
    }
    float* out = a.ws_partial + ((head0 + h) * (size_t)n_slots + slot) * (D + 2);
    if (c == 0) store_device(out, m_ref[h], den);
    store_device(out + 2 + c, num[0], num[1]);
  }
  if (n_slots == 1) return;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  const size_t at = row * a.sets + set;
  if (threadIdx.x == 0)
    s_last = (ROW ? count_in(a.ws_tags + at, a.tag, seen)
                  : __hip_atomic_fetch_add(a.ws_count + at, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == n_slots - 1;
  __syncthreads();
  if (!s_last) return;
  merge_partials<D, kWaves>(a.ws_partial + head0 * n_slots * (D + 2), n_slots, gh, a.out + head0 * D, nullptr, threadIdx.x);
  // nobody looks at these any more; a replay of a recorded launch starts from here
  if constexpr (ROW) {
    for (int i = threadIdx.x; i < gh * a.cb * 2; i += kThreads) a.ws_words[head0 * a.cb * 2 + i] = 0;
    if (threadIdx.x == 0) a.ws_tags[at] = 0;
  }
}

// Tokens t0 .. t1 of the fp16 tail: weights in fp32 (lane = token), then lane = (token slot, channel octet).
// lg: logit of the set's first head and token base, pitch floats between two heads.  ready(m_ref), called behind the
// first loads, leaves the logits in lg and the reference point of every head in m_ref.
template <int D, bool ROW, typename Ready>
__device__ inline void text_values(const TileArgs& a, size_t row, int set, int t0, int t1, int slot, u64 seen, int lane,
                                   int wave, const float* lg, size_t pitch, int base, float (*s_p)[kHeads],
                                   float (*s_part)[kHeads][D], float (*s_lm)[kHeads][2], Ready ready) {
  constexpr int kOct = D / 8, kSlots = 64 / kOct;
  const int gh = min(kHeads, a.g - set * kHeads);
  const size_t head0 = row * a.g + (size_t)set * kHeads;
  const __half* vals = a.v_text + row * (size_t)a.n_text_cap * D;
  const int c8 = lane & (kOct - 1), ts = lane / kOct;
  constexpr int kLoads = kTextShare / kSlots;                  // a share's loads are in flight together
  v8h v[kLoads];
  auto load_share = [&](int t) {               // past the end: the last token, which gets weight 0
#pragma unroll
    for (int i = 0; i < kLoads; ++i)
      v[i] = *reinterpret_cast<const v8h*>(vals + (size_t)min(t + i * kSlots + ts, t1 - 1) * D + 8 * c8);
  };
  const int first = t0 + kTextShare * wave;
  constexpr bool kEarly = D == 64;             // (registers)
  if (kEarly && first < t1) load_share(first);
  float m_ref[kHeads], l[kHeads], acc[kHeads][8];
  ready(m_ref);
#pragma unroll
  for (int h = 0; h < kHeads; ++h) {
    if (t1 <= t0) m_ref[h] = -FLT_MAX;         // an empty chunk has weight 0
    l[h] = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[h][j] = 0.f;
  }
  for (int t = first; t < t1; t += kTextBlock) {
    const int nt = min(kTextShare, t1 - t);
    if (!kEarly) load_share(t);
    v4f p = {0.f, 0.f, 0.f, 0.f};
    if (lane < nt) {
#pragma unroll
      for (int h = 0; h < kHeads; ++h)
        if (h < gh) p[h] = __builtin_amdgcn_exp2f((lg[h * pitch + (t - base) + lane] - m_ref[h]) * kLog2e);
    }
#pragma unroll
    for (int h = 0; h < kHeads; ++h) l[h] += p[h];
    __builtin_amdgcn_wave_barrier();
    if (lane < kTextShare) *reinterpret_cast<v4f*>(s_p[kTextShare * wave + lane]) = p;
    lds_publish();
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const v4f w = *reinterpret_cast<const v4f*>(s_p[kTextShare * wave + i * kSlots + ts]);
#pragma unroll
      for (int h = 0; h < kHeads; ++h)
#pragma unroll
        for (int u = 0; u < 8; ++u) acc[h][u] = fmaf(w[h], (float)v[i][u], acc[h][u]);
    }
    __builtin_amdgcn_wave_barrier();
    if (kEarly && t + kTextBlock < t1) load_share(t + kTextBlock);
  }
  // sum over the token slots; the paired folds leave one head per half or row of the wave
  if constexpr (D == 256) {                    // two slots: lanes 0-31 and 32-63
    float r[2][8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      r[0][u] = fold_halves(acc[0][u], acc[1][u]);
      r[1][u] = fold_halves(acc[2][u], acc[3][u]);
    }
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int u = 0; u < 8; u += 4)
        *reinterpret_cast<v4f*>(&s_part[wave][2 * e + (lane >> 5)][8 * c8 + u]) =
            (v4f){r[e][u], r[e][u + 1], r[e][u + 2], r[e][u + 3]};
  } else {                                     // four slots (rows of 16 lanes), or eight (half rows)
    float r[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if constexpr (D == 64) {
#pragma unroll
        for (int h = 0; h < kHeads; ++h) acc[h][u] += dpp_f32<0x128>(acc[h][u]);     // row_ror 8
      }
      r[u] = fold_rows(fold_halves(acc[0][u], acc[2][u]), fold_halves(acc[1][u], acc[3][u]));
    }
    if (D == 128 || (lane & 8) == 0) {
#pragma unroll
      for (int u = 0; u < 8; u += 4)
        *reinterpret_cast<v4f*>(&s_part[wave][lane >> 4][8 * c8 + u]) = (v4f){r[u], r[u + 1], r[u + 2], r[u + 3]};
    }
  }
  const float lw = head_sums(l, lane);
  if ((lane & 15) == 0) { s_lm[wave][lane >> 4][0] = lw; s_lm[wave][lane >> 4][1] = 0.f; }
  finish_chunk<D, ROW>(a, row, set, head0, gh, slot, seen, m_ref, s_part, s_lm);
}
__device__ inline int text_length(const TileArgs& a) {
  return a.n_text_dev ? min(max(*a.n_text_dev, 0), a.n_text) : a.n_text;
}

// What a wave of the values pass stages, and what the workgroup's waves leave for its end.
template <int D, int BITS>
struct ValueLds {
  static constexpr int CB = D * BITS / 8;                      // code bytes per token
  static constexpr int SW = CB < 128 ? CB : 128;               // bytes per token staged at a time
  static constexpr int kPitch = SW >= 64 ? SW + 16 : SW;       // spreads the transposing reads over the banks
  struct Stage { uint8_t x[1024]; uint8_t codes[64 * kPitch]; };
  union Mem {
    Stage stage[kWaves];
    float part[kWaves][kHeads][D];
    uint8_t key_operand[kWaves][Operand<D, BITS>::kProducts * 1024];     // tile_row_kernel: before the values
  };
};

// Value tiles u0 .. u1 of a row: weights and values, one partial of the joint softmax.  logits: of the set's first
// head and token base, pitch floats between two heads (ROW: in LDS).  extrema(lo, hi), called behind the first loads,
// gives lane row h those of head h; false: not yet, the workgroup has to form them itself.
template <int D, int BITS, bool VCH, bool ROW, typename Extrema>
__device__ inline bool visual_values(const TileArgs& a, size_t row, int set, int u0, int u1, int slot, u64 seen, int lane,
                                     int wave, const float* logits, size_t pitch, int base,
                                     typename ValueLds<D, BITS>::Mem& mem, float (*s_lm)[kHeads][2], Extrema extrema) {
  constexpr int CB = D * BITS / 8;                             // code bytes per token
  constexpr int kV = 8 / BITS;
  constexpr int kBlocks = CB >= 16 ? CB / 16 : 1;              // 16-byte column blocks (8 bytes: half of one)
  constexpr int NACC = kBlocks * kV;
  constexpr int SW = ValueLds<D, BITS>::SW, kPitch = ValueLds<D, BITS>::kPitch;
  constexpr int kPasses = CB / SW;
  constexpr int kPieces = SW >= 16 ? SW / 16 : 1;              // 16-byte (8-byte) loads per lane and pass
  constexpr int kPieceBytes = SW >= 16 ? 16 : 8;
  const int n16 = lane & 15, kb = lane >> 4;
  const int gh = min(kHeads, a.g - set * kHeads);
  const size_t head0 = row * a.g + (size_t)set * kHeads;

  // the wave's run of tiles
  const int per = (u1 - u0) / kWaves, rem = (u1 - u0) % kWaves;
  const int k0 = u0 + chunk_first(per, rem, wave), k1 = u0 + chunk_first(per, rem, wave + 1);

  const uint8_t* vc = reinterpret_cast<const uint8_t*>(a.v_codes) + row * (size_t)a.n_vis * CB;
  const float* vs = a.v_scale + row * (size_t)a.n_vis;         // token-wise
  const uint16_t* vm = a.v_min + row * (size_t)a.n_vis;
  const size_t meta0 = VCH ? row * (size_t)a.v_groups * D : 0;
  const float* lg[kHeads];
#pragma unroll
  for (int h = 0; h < kHeads; ++h) lg[h] = logits + min(h, gh - 1) * pitch;
  uint8_t* xbuf = mem.stage[wave].x;
  uint8_t* cbuf = mem.stage[wave].codes;
  const uint8_t* x_rd = xbuf + (kb * 16 + (n16 >> 1)) * 16 + (n16 & 1) * 8;
  // (8-byte tokens: the upper eight columns repeat the lower eight and are dropped at the end)
  const uint8_t* v_rd = cbuf + (kb * 16 + (n16 >> 1)) * kPitch + (CB >= 16 ? (n16 & 1) * 8 : 0);
  // channel of accumulator p (column block cb, variant v) in this lane
  auto channel = [&](int p) {
    const int tb = 16 * (p / kV) + (CB >= 16 ? n16 : n16 & 7);
    return (32 / BITS) * (tb >> 2) + code_in_word<BITS>(tb & 3, p % kV);
  };

  v4i acc[NACC], acc_w = {0, 0, 0, 0};
  float facc[NACC], lsum[kHeads], msum[kHeads];
#pragma unroll
  for (int p = 0; p < NACC; ++p) { acc[p] = (v4i){0, 0, 0, 0}; facc[p] = 0.f; }
#pragma unroll
  for (int h = 0; h < kHeads; ++h) lsum[h] = msum[h] = 0.f;
  // What goes into the matrix product is w = p (channel-wise values) or p * scale (token-wise), as the
  // integer nearest to w times a power of two.  That scale is a head's own and follows the products, not
  // the tokens' scales: the largest w so far of the head is in [2^25, 2^29), so no bits are spent on a
  // token that stands out but that the head does not look at, nor on what another head looks at.  It
  // only drops, within a channel-wise group (whose parameters are its own).  Where the group is the whole
  // row all weights meet the same parameters and the largest is 1: 2^28 throughout, as weights far below
  // count for nothing.
  Scales scales(VCH && a.v_groups == 1 ? 28 : 90);
  int run = 0;

  v4i piece_r[kPieces];
  float lgv[kHeads], sc = 0.f;
  uint16_t mi = 0;
  float gs[VCH ? NACC : 1];                                    // channel-wise: parameters of group `params_of`
  uint16_t gm[VCH ? NACC : 1];
  int params_of = -1;
  auto tile_at = [&](int k, int& grp, int& tok0, int& nt) {
    grp = part_of(k, a.v_tpg);
    const int sub = k - grp * a.v_tpg;
    tok0 = grp * a.v_group + sub * kValTile;
    nt = min(kValTile, a.v_group - sub * kValTile);
  };
  auto load_pieces = [&](int tok0, int nt, int pass) {
    const uint8_t* base = vc + (size_t)tok0 * CB + pass * SW;
#pragma unroll
    for (int e = 0; e < kPieces; ++e) {
      const int o = 64 * kPieceBytes * e + kPieceBytes * lane;
      const uint8_t* p = base + (size_t)min(o / SW, nt - 1) * CB + o % SW;
      if constexpr (kPieceBytes == 16) {
        piece_r[e] = *reinterpret_cast<const v4i*>(p);
      } else {
        const v2i t = *reinterpret_cast<const v2i*>(p);
        piece_r[e] = (v4i){t[0], t[1], 0, 0};
      }
    }
  };
  auto load_tile = [&](int k) {
    int grp, tok0, nt;
    tile_at(k, grp, tok0, nt);
    const int j = tok0 + min(lane, nt - 1);
    if constexpr (!ROW) {
#pragma unroll
      for (int h = 0; h < kHeads; ++h) lgv[h] = lg[h][j - base];
    }
    if constexpr (!VCH) {
      sc = vs[j];
      mi = vm[j];
    }
    load_pieces(tok0, nt, 0);
  };
  auto load_params = [&](int grp) {
    params_of = grp;
    if constexpr (VCH) {
#pragma unroll
      for (int p = 0; p < NACC; ++p) {
        const size_t at = meta0 + (size_t)grp * D + channel(p);
        gs[p] = a.v_scale[at];
        gm[p] = a.v_min[at];
      }
    }
  };
  // the first tile is asked for before the extrema are folded, so that a wave waits for memory once
  if (k0 < k1) {
    load_tile(k0);
    load_params(part_of(k0, a.v_tpg));
  }
  // ---- calibration line and reference point per head (Sec. 3.2)
  float a2[kHeads], c2[kHeads], m_ref[kHeads];
  {
    float lo_l, hi_l;
    if (!extrema(lo_l, hi_l)) return false;
    // (the lanes of row h work on head h: one division for all four)
    float slope = 1.f, gam = 0.f, shift = 0.f;                 // s' = slope * (s - gam) + shift
    if (a.calib_mode != CQ_CALIB_NONE) {
      const float glo = a.calib_mode == CQ_CALIB_DYNAMIC ? lo_l : a.gamma;
      const float ghi = a.calib_mode == CQ_CALIB_DYNAMIC ? hi_l : a.delta;
      const float width = ghi - glo;
      slope = width == 0.f ? 1.f : (width + a.tau1 - a.tau2) / width;
      gam = glo;
      shift = glo - a.tau1;
    }
    // the map is monotone: an end of the row's range is its maximum, every weight is <= 1
    const float M = fmaxf(slope * (lo_l - gam) + shift, slope * (hi_l - gam) + shift);
    const float c = (shift - slope * gam - M) * kLog2e;
#pragma unroll
    for (int h = 0; h < kHeads; ++h) {
      m_ref[h] = lane_value(M, 16 * h);
      a2[h] = h < gh ? lane_value(slope, 16 * h) * kLog2e : 0.f;
      c2[h] = h < gh ? lane_value(c, 16 * h) : -200.f;         // no head: weight 0
    }
  }

  // the digit sums into fp32, weighted (channel-wise: by the parameters of the group they belong to)
  auto bank = [&]() {
    const float unit = scales.inverse(kb);
    const float wsum = VCH ? digits_to_float(acc_w) * unit : 0.f;
    acc_w = (v4i){0, 0, 0, 0};
#pragma unroll
    for (int p = 0; p < NACC; ++p) {
      const float sum = digits_to_float(acc[p]) * unit;
      acc[p] = (v4i){0, 0, 0, 0};
      if constexpr (VCH) {
        const float add = __half2float(__ushort_as_half(gm[p])) + (BITS == 8 ? 128.f * gs[p] : 0.f);
        facc[p] = fmaf(sum, gs[p] * variant_weight<BITS>(p % kV), fmaf(wsum, add, facc[p]));
      } else {
        facc[p] += sum;
      }
    }
    run = 0;
  };

  for (int k = k0; k < k1; ++k) {
    int grp, tok0, nt;
    tile_at(k, grp, tok0, nt);
    if constexpr (ROW) {                       // (on chip: read when they are needed)
      const int j = tok0 + min(lane, nt - 1);
#pragma unroll
      for (int h = 0; h < kHeads; ++h) lgv[h] = lg[h][j - base];
    }
    const bool have = lane < nt, next_group = VCH && grp != params_of;         // (the latter wave-uniform)
    float w[kHeads], x[kHeads];
#pragma unroll
    for (int h = 0; h < kHeads; ++h) {
      const float e = __builtin_amdgcn_exp2f(fmaf(lgv[h], a2[h], c2[h]));
      const float p = have ? e : 0.f;
      lsum[h] += p;
      if constexpr (VCH) {
        w[h] = p;
      } else {
        w[h] = p * sc;
        msum[h] = fmaf(p, __half2float(__ushort_as_half(mi)) + (BITS == 8 ? 128.f * sc : 0.f), msum[h]);
      }
      x[h] = digits_bias(w[h], scales.of(h));
    }
    auto bits_of = [](float v) { return __builtin_bit_cast(int, v); };
    const bool over = max(max(bits_of(x[0]), bits_of(x[1])), max(bits_of(x[2]), bits_of(x[3]))) >= bits_of(0x1p29f);
    if (__builtin_amdgcn_ballot_w64(over) != 0 || run == kMaxRun || next_group) {
      if (run) bank();           // the four digit sums of a value cannot be scaled one by one
      if (next_group) {
        load_params(grp);
        scales = Scales(90);
      }
      scales.lower(w, lane);
#pragma unroll
      for (int h = 0; h < kHeads; ++h) x[h] = digits_bias(w[h], scales.of(h));
    }
    v4i xs;
#pragma unroll
    for (int h = 0; h < kHeads; ++h) xs[h] = (int)x[h] ^ 0x00808080;
    __builtin_amdgcn_wave_barrier();
    *reinterpret_cast<v4i*>(xbuf + 16 * lane) = xs;
    v4i A;
#pragma unroll
    for (int pass = 0; pass < kPasses; ++pass) {
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int e = 0; e < kPieces; ++e) {
        const int o = 64 * kPieceBytes * e + kPieceBytes * lane;
        uint8_t* dst = cbuf + (o / SW) * kPitch + o % SW;
        if constexpr (kPieceBytes == 16) *reinterpret_cast<v4i*>(dst) = piece_r[e];
        else *reinterpret_cast<v2i*>(dst) = (v2i){piece_r[e][0], piece_r[e][1]};
      }
      lds_publish();
      if (pass == 0) {
        const v2i lo = lds_read_tr8(x_rd), hi = lds_read_tr8(x_rd + 128);
        A = (v4i){lo[0], lo[1], hi[0], hi[1]};
      }
      // the next loads go out under the products
      if (pass + 1 < kPasses) load_pieces(tok0, nt, pass + 1);
      else if (k + 1 < k1) load_tile(k + 1);
      constexpr int kPassBlocks = SW >= 16 ? SW / 16 : 1;
#pragma unroll
      for (int cbl = 0; cbl < kPassBlocks; ++cbl) {
        const v2i lo = lds_read_tr8(v_rd + 16 * cbl), hi = lds_read_tr8(v_rd + 16 * cbl + 8 * kPitch);
        const v4i raw = {lo[0], lo[1], hi[0], hi[1]};
#pragma unroll
        for (int v = 0; v < kV; ++v) {
          v4i B;
#pragma unroll
          for (int u = 0; u < 4; ++u) B[u] = operand_variant<BITS>((uint32_t)raw[u], v);
          const int p = (pass * kPassBlocks + cbl) * kV + v;
          acc[p] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A, B, acc[p], 0, 0, 0);
        }
      }
    }
    ++run;
    if constexpr (VCH) {
      const v4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
      acc_w = __builtin_amdgcn_mfma_i32_16x16x64_i8(A, ones, acc_w, 0, 0, 0);
    }
  }
  if (run) bank();
  __syncthreads();                                             // the stages become the partial sums
#pragma unroll
  for (int p = 0; p < NACC; ++p) {
    const float v = VCH ? facc[p] : facc[p] * variant_weight<BITS>(p % kV);
    if (CB >= 16 || n16 < 8) mem.part[wave][kb][channel(p)] = v;
  }
  const float l = head_sums(lsum, lane), m = head_sums(msum, lane);      // of head kb
  if (n16 == 0) { s_lm[wave][kb][0] = l; s_lm[wave][kb][1] = m; }
  finish_chunk<D, ROW>(a, row, set, head0, gh, slot, seen, m_ref, mem.part, s_lm);
  return true;
}

// grid: x = row, y = chunk of the tail, then chunk of the visual tokens, z = head set
template <int D, int BITS, bool VCH>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(D == 256 || BITS == 8 ? 2 : D == 128 && BITS >= 2 && VCH ? 3 : 4)))
tile_values_kernel(const TileArgs a) {
  __shared__ __align__(16) typename ValueLds<D, BITS>::Mem mem;
  __shared__ __align__(16) float s_lm[kWaves][kHeads][2];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const size_t row = blockIdx.x;
  const int set = (int)blockIdx.z, chunk = (int)blockIdx.y - a.ct;
  const int gh = min(kHeads, a.g - set * kHeads);
  const size_t head0 = row * a.g + (size_t)set * kHeads, n_all = (size_t)a.n_vis + a.n_text;
  if (chunk < 0) {
    __shared__ __align__(16) float s_tp[kTextBlock][kHeads];
    const int t0 = (int)blockIdx.y * a.ct_tokens, t1 = min(t0 + a.ct_tokens, text_length(a));
    text_values<D, false>(a, row, set, t0, t1, a.cb + (int)blockIdx.y, 0, lane, wave, a.ws_logits + head0 * n_all + a.n_vis,
                   n_all, 0, s_tp, mem.part, s_lm, [&](float (&m_ref)[kHeads]) {
#pragma unroll
      for (int h = 0; h < kHeads; ++h)
        m_ref[h] = a.ws_minmax[((head0 + min(h, gh - 1)) * (size_t)(a.ca + a.ct) + a.ca + blockIdx.y) * 2 + 1];
    });
    return;
  }
  const int u0 = chunk_first(a.cb_base, a.cb_rem, chunk), u1 = chunk_first(a.cb_base, a.cb_rem, chunk + 1);
  visual_values<D, BITS, VCH, false>(a, row, set, u0, u1, chunk, 0, lane, wave, a.ws_logits + head0 * n_all, n_all, 0, mem,
                                     s_lm, [&](float& lo, float& hi) {
    // lane 16 h + c folds chunks c, c + 16, ... of head h
    const float* mm = a.ws_minmax + (head0 + min(lane >> 4, gh - 1)) * (size_t)(a.ca + a.ct) * 2;
    lo = FLT_MAX;
    hi = -FLT_MAX;
    for (int c = lane & 15; c < a.ca; c += 16) {
      lo = fminf(lo, mm[2 * c]);
      hi = fmaxf(hi, mm[2 * c + 1]);
    }
    lo = row_min(lo);
    hi = row_max(hi);
    return true;
  });
}

// ===================================================================================== one launch
// The logits of a chunk of visual tokens stay in LDS, the workgroups of a row exchange their extrema
// (decode_meet.h); a chunk of the tail needs nothing from anybody.  Against the two launches above it saves the
// second one's start, the round trip of the logits through memory and the tail's second query: 64 rows x 3003
// tokens, 2 bits, whole-sequence keys and values 15.5 -> 13.2 us, 8 such rows 11.5 -> 10.3, 16 rows x 3328 tokens of
// 256 channels 12.2 -> 11.3, 256 rows x 8001 55.2 -> 47.6.
// grid: the slots of a (row, head set) one after the other, chunks of the tail first
extern __shared__ __align__(16) float s_logits[];              // [kHeads][l_stride]
template <int D, int BITS, bool VCH>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(D == 256 || BITS == 8 ? 2 : D == 128 && BITS >= 2 && VCH ? 3 : 4)))
tile_row_kernel(const TileArgs args) {
  __shared__ __align__(16) typename ValueLds<D, BITS>::Mem mem;
  __shared__ __align__(16) float s_lm[kWaves][kHeads][2];
  __shared__ float red[kWaves][kHeads][2];
  __shared__ float s_row[kHeads][2];
  __shared__ int s_found;
  float row_lo = FLT_MAX, row_hi = -FLT_MAX;                   // lane row h: extrema of head h, passes so far
  u64 seen = 0;
  // one pass over the workgroup's own chunk; if the others' extrema do not turn up, one over each of theirs
  for (int pass = 0;; ++pass) {
    int tid = threadIdx.x;                     // (arguments and lane out of the compiler's sight: see decode_fused.hip)
    auto kernarg = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+v"(tid), "+s"(kernarg));
    const TileArgs& a = *(const TileArgs*)kernarg;
    // the arguments' cache lines, together
    asm volatile("" :: "s"(a.q), "s"(a.k_text), "s"(a.k_group), "s"(a.l_stride), "s"(a.patience));
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n16 = lane & 15, kb = lane >> 4;
    const int n_slots = a.cb + a.ct;
    const int rs = a.slots_magic ? (int)__umulhi((unsigned)blockIdx.x, a.slots_magic) : (int)blockIdx.x;
    const int slot = (int)blockIdx.x - rs * n_slots;
    const size_t row = a.sets == 1 ? rs : rs / a.sets;
    const int set = a.sets == 1 ? 0 : rs % a.sets;
    const int gh = min(kHeads, a.g - set * kHeads);
    const size_t head0 = row * a.g + (size_t)set * kHeads;
    if (pass == 0 && tid == 0 && n_slots > 1) seen = count_open(a.ws_tags + row * a.sets + set, a.tag);
    if (slot < a.ct) {
      __shared__ __align__(16) float s_tp[kTextBlock][kHeads];
      const int t0 = slot * a.ct_tokens, t1 = min(t0 + a.ct_tokens, text_length(a));
      text_values<D, true>(a, row, set, t0, t1, slot, seen, lane, wave, s_logits, a.l_stride, t0, s_tp, mem.part, s_lm,
                     [&](float (&m_ref)[kHeads]) {
        // the logits of the shares that this wave weights, on the fp16 matrix cores as in text_logits
        v8h A[D / 32];
#pragma unroll
        for (int s = 0; s < D / 32; ++s)       // (matrix rows from gh on repeat the last head)
          A[s] = *reinterpret_cast<const v8h*>(a.q + (head0 + min(n16, gh - 1)) * D + 32 * s + 8 * kb);
        float mx[kHeads];
#pragma unroll
        for (int h = 0; h < kHeads; ++h) mx[h] = -FLT_MAX;
        const __half* keys = a.k_text + row * (size_t)a.n_text_cap * D + 8 * kb;
        constexpr int kFly = kTextShare / 16;
        for (int t = t0 + kTextShare * wave; t < t1; t += kTextBlock) {
          v8h kv[kFly][D / 32];
#pragma unroll
          for (int u = 0; u < kFly; ++u)
#pragma unroll
            for (int s = 0; s < D / 32; ++s)
              kv[u][s] = *reinterpret_cast<const v8h*>(keys + (size_t)min(t + 16 * u + n16, t1 - 1) * D + 32 * s);
#pragma unroll
          for (int u = 0; u < kFly; ++u) {
            v4f c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < D / 32; ++s) c = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[s], kv[u][s], c, 0, 0, 0);
            if (kb == 0) {                     // result rows 0..3; past the end: the last token again
#pragma unroll
              for (int h = 0; h < kHeads; ++h) {
                const float x = c[h] * a.softmax_scale;
                s_logits[h * a.l_stride + t - t0 + 16 * u + n16] = x;
                mx[h] = fmaxf(mx[h], x);
              }
            }
          }
        }
#pragma unroll
        for (int h = 0; h < kHeads; ++h) {
          const float m = row_max(mx[h]);
          if (lane == 0) red[wave][h][1] = m;
        }
        __syncthreads();
#pragma unroll
        for (int h = 0; h < kHeads; ++h) {
          m_ref[h] = red[0][h][1];
#pragma unroll
          for (int w = 1; w < kWaves; ++w) m_ref[h] = fmaxf(m_ref[h], red[w][h][1]);
        }
      });
      return;
    }
    const int own = slot - a.ct;
    int chunk = own + pass;
    if (chunk >= a.cb) chunk -= a.cb;
    const int u0 = chunk_first(a.cb_base, a.cb_rem, chunk), u1 = chunk_first(a.cb_base, a.cb_rem, chunk + 1);
    if (pass <= a.cb - 1) {                    // (pass cb: all extrema are known, the logits in place)
      float mn = FLT_MAX, mx = -FLT_MAX;
      visual_logits<D, BITS>(a, row, set, min(u0 * a.k_bpu, a.k_blocks), min(u1 * a.k_bpu, a.k_blocks), lane, wave,
                             mem.key_operand[wave], chunk == own, s_logits + kb * a.l_stride, u0 * kUnit, mn, mx);
      mn = row_min(mn);
      mx = row_max(mx);
      __builtin_amdgcn_wave_barrier();
      if (n16 == 0) {
        red[wave][kb][0] = mn;
        red[wave][kb][1] = mx;
      }
      __syncthreads();
      row_lo = fminf(row_lo, row_min(red[n16 & (kWaves - 1)][kb][0]));
      row_hi = fmaxf(row_hi, row_max(red[n16 & (kWaves - 1)][kb][1]));
      if (pass > 0) { __syncthreads(); continue; }
      // stored now: what comes before the others' are needed hides the way there
      if (a.calib_mode == CQ_CALIB_DYNAMIC && a.cb > 1 && wave == 0 && n16 == 0 && kb < gh)
        post_extrema(a.ws_words + ((head0 + kb) * (size_t)a.cb + own) * 2, row_lo, row_hi, a.tag);
    }
    const bool done = visual_values<D, BITS, VCH, true>(
        a, row, set, min(u0 * a.v_tpu, a.v_tiles), min(u1 * a.v_tpu, a.v_tiles), slot, seen, lane, wave,
        s_logits, a.l_stride, u0 * kUnit, mem, s_lm, [&](float& lo, float& hi) {
      lo = row_lo;
      hi = row_hi;
      if (a.calib_mode != CQ_CALIB_DYNAMIC || a.cb == 1 || pass > 0) return true;
      if (wave == 0) {
        const u64* words = a.ws_words + (head0 + min(kb, gh - 1)) * (size_t)a.cb * 2;
        float all_lo = FLT_MAX, all_hi = -FLT_MAX;
        bool all = false;
        for (int look = 0; !all && look < a.patience; ++look) {
          all_lo = lo;
          all_hi = hi;
          all = true;
          for (int c = n16; c < a.cb; c += 16) {
            if (c == own) continue;
            float x, y;
            all = read_extrema(words + 2 * c, &x, &y, a.tag) && all;
            all_lo = fminf(all_lo, x);
            all_hi = fmaxf(all_hi, y);
          }
          all = __builtin_amdgcn_ballot_w64(!all) == 0;
          if (!all) __builtin_amdgcn_s_sleep(1);
        }
        all_lo = row_min(all_lo);
        all_hi = row_max(all_hi);
        if (n16 == 0) {
          s_row[kb][0] = all_lo;
          s_row[kb][1] = all_hi;
        }
        if (lane == 0) s_found = all;
      }
      __syncthreads();
      if (!s_found) { __syncthreads(); return false; }
      lo = s_row[kb][0];
      hi = s_row[kb][1];
      return true;
    });
    if (done) return;
  }
}

using TileKernel = void (*)(const TileArgs);

template <int D>
TileKernel logits_kernel(int bits) {
  switch (bits) {
    case 1: return tile_logits_kernel<D, 1>;
    case 2: return tile_logits_kernel<D, 2>;
    case 4: return tile_logits_kernel<D, 4>;
    case 8: return tile_logits_kernel<D, 8>;
    default: return nullptr;
  }
}
template <int D>
TileKernel values_kernel(int bits, bool vch) {
  switch (bits * 2 + (vch ? 1 : 0)) {
    case 2: return tile_values_kernel<D, 1, false>;
    case 3: return tile_values_kernel<D, 1, true>;
    case 4: return tile_values_kernel<D, 2, false>;
    case 5: return tile_values_kernel<D, 2, true>;
    case 8: return tile_values_kernel<D, 4, false>;
    case 9: return tile_values_kernel<D, 4, true>;
    case 16: return tile_values_kernel<D, 8, false>;
    case 17: return tile_values_kernel<D, 8, true>;
    default: return nullptr;
  }
}

template <int D>
TileKernel row_kernel(int bits, bool vch) {
  switch (bits * 2 + (vch ? 1 : 0)) {
    case 2: return tile_row_kernel<D, 1, false>;
    case 3: return tile_row_kernel<D, 1, true>;
    case 4: return tile_row_kernel<D, 2, false>;
    case 5: return tile_row_kernel<D, 2, true>;
    case 8: return tile_row_kernel<D, 4, false>;
    case 9: return tile_row_kernel<D, 4, true>;
    case 16: return tile_row_kernel<D, 8, false>;
    case 17: return tile_row_kernel<D, 8, true>;
    default: return nullptr;
  }
}

}  // namespace

namespace {

// One launch where chunks of whole units can be made of whole key blocks and value tiles, and their logits take
// little enough LDS for several workgroups per CU.  It is faster on small calls of every head_dim (100 drawn
// layouts below 100 thousand tokens: 1.06 with 64 channels, 1.2 with 128, 1.17 with 256) and with 128 channels on large
// ones too (1.3 beyond 600 thousand).  With 64 and 256 channels and with 8 bits it is not: all workgroups pass the exchange
// together, so memory and matrix cores idle in turn (64 rows of 64 channels x 3328 tokens, two / one: 13.6 / 12.8 us,
// x 8192 17.9 / 18.5; 480 rows of 256 channels x 4352 77 / 99; 144 x 1198, 4 bits 25.3 / 30.1), the more so in key groups of
// 32, and with 256 channels, 8 bits, or 64 channels of few rows in groups of 64, which leave a wave short blocks (128 x 640, 6
// heads, 2 bits, 256 channels 17.4 / 25.0; 16 x 1536, 8 bits 12.1 / 13.9; 8 x 3328, 4 bits, 64 channels 9.5 / 10.9; but 157 x
// 256, 8 bits 15.3 / 13.0; and without a calibration range to find there is no exchange: 32 x 1472, 1 bit, 64 channels
// 10.2 / 9.3).  768 workgroups: three per CU are resident whatever the registers (256 rows x 2001, 1024 / 768:
// 21.3 / 18.6); chunks below four units only lengthen the exchange and the merge (64 rows x 3003: 23.6 us with
// two, 14.9 with four), and more than 56 chunks of a row cost more than they save (8 rows x 60608 25.8 / 31.2).
void plan_one_launch(const DecodeShape& s, long long rows, long long sets, TilePlan* p) {
  auto fits_units = [&](int axis, int group) {
    return axis != CQ_AXIS_CHANNEL || group == s.n_vis || group % kUnit == 0 || kUnit % group == 0;
  };
  const int units = ceil_div(s.n_vis, kUnit);
  p->row_ct = p->ct;
  if (s.k_group < 64 && s.k_group != s.n_vis) return;
  if ((s.d != 128 || s.bits == 8) && (s.n_vis > kRowMost || rows * sets * s.n_vis > kRowMostAll)) return;
  const bool exchange_pays = !(s.d == 256 && rows * sets * s.n_vis > kRowMostWide) &&
                             !(s.k_group == 64 && s.n_vis > kRowMostShort &&
                               (s.d == 256 || s.bits == 8 || (s.d == 64 && rows * sets * s.n_vis < kRowLeast64)));
  if (s.n_vis > 0) {
    if (!fits_units(s.k_axis, s.k_group) || !fits_units(s.v_axis, s.v_group)) return;
    const long long want = (kRowTarget + rows * sets - 1) / (rows * sets);
    const int least = ceil_div(units, kRowMaxUnits), most = ceil_div(units, kRowMinUnits);
    if (least > kRowMostChunks) return;
    p->row_cb = (int)(want < least ? least : want > most ? most : want);
    if (p->row_cb > kRowMostChunks) p->row_cb = kRowMostChunks;
  }
  if (p->ct_tokens > kRowMaxUnits * kUnit) return;
  const long long slots = p->row_cb + p->row_ct;
  if (slots < 1 || rows * sets * slots * slots >= (1LL << 32)) return;
  auto align64 = [](size_t x) { return (x + 63) / 64 * 64; };
  const size_t heads = (size_t)s.B * s.Hq;
  p->row_tags_floats = align64(heads * (size_t)p->row_cb * 4);
  p->row_partial_floats = align64(p->row_tags_floats + (size_t)(rows * sets) * 2);
  const size_t floats = p->row_partial_floats + heads * (size_t)slots * (s.d + 2);
  p->one_launch_free = floats * sizeof(float) <= p->ws_bytes;
  p->one_launch = p->one_launch_free && exchange_pays;
}

}  // namespace

TilePlan make_tile_plan(const DecodeShape& s, size_t limit) {
  TilePlan p;
  if (s.d != 64 && s.d != 128 && s.d != 256) return p;
  if (s.bits != 1 && s.bits != 2 && s.bits != 4 && s.bits != 8) return p;
  if (s.k_axis != CQ_AXIS_CHANNEL) return p;
  if (s.v_axis != CQ_AXIS_CHANNEL && s.v_group != s.d) return p;
  const long long rows = (long long)s.B * s.Hkv, sets = (s.g + kHeads - 1) / kHeads;
  auto clamp = [](long long v, long long lo, long long hi) { return (int)(v < lo ? lo : v > hi ? hi : v); };
  if (s.n_vis > 0) {
    const long long blocks = (long long)(s.n_vis / s.k_group) * ceil_div(s.k_group, kKeyBlock);
    const long long tiles = s.v_axis == CQ_AXIS_CHANNEL
                                ? (long long)(s.n_vis / s.v_group) * ceil_div(s.v_group, kValTile)
                                : ceil_div(s.n_vis, kValTile);
    // four workgroups per CU, of at least one key block (two value tiles) per wave
    const long long want = (1024 + rows * sets - 1) / (rows * sets);
    p.ca = clamp(want, 1, clamp((blocks + kWaves - 1) / kWaves, 1, kMaxTileChunks));
    p.cb = clamp(want, 1, clamp((tiles + 2 * kWaves - 1) / (2 * kWaves), 1, kMaxTileChunks));
  }
  // the tail does not change how the visual tokens are divided
  p.ct_tokens = kTextBlock * ceil_div(ceil_div(s.n_text, kTextBlock), kMaxTileChunks);
  if (s.n_text > 0) p.ct = ceil_div(s.n_text, p.ct_tokens);
  const size_t heads = (size_t)s.B * s.Hq;
  auto align64 = [](size_t x) { return (x + 63) / 64 * 64; };
  auto lay_out = [&](int ct) {
    p.ws_minmax_floats = align64(heads * ((size_t)s.n_vis + s.n_text));
    p.ws_partial_floats = align64(p.ws_minmax_floats + heads * (size_t)(p.ca + ct) * 2);
    p.ws_count_floats = align64(p.ws_partial_floats + heads * (size_t)(p.cb + ct) * (s.d + 2));
    return ((p.ws_count_floats + (size_t)(rows * sets)) * sizeof(float) + 255) / 256 * 256;
  };
  // Where the chunks of the tail grow their number falls, from 64 to 33 past 8192 tokens.  What a caller
  // is asked for does not: it counts the most chunks that a tail of up to n_text tokens is cut into, so
  // that a workspace for a longer tail serves a shorter one.
  const int text_blocks = ceil_div(s.n_text, kTextBlock);
  p.ws_reserve_bytes = lay_out(text_blocks < kMaxTileChunks ? text_blocks : kMaxTileChunks);
  p.ws_bytes = lay_out(p.ct);
  // within the limit: fewer chunks, of whichever kind has more of them
  bool fits = true;
  while (p.ws_bytes > limit && fits) {
    if (p.ct > 1 && (p.ct >= p.cb || p.cb <= 1)) {
      p.ct_tokens = kTextBlock * ceil_div(text_blocks, p.ct - 1);
      p.ct = ceil_div(s.n_text, p.ct_tokens);
    } else if (p.cb > 1) {
      --p.cb;
    } else {
      fits = false;
    }
    p.ws_bytes = lay_out(p.ct);
  }
  plan_one_launch(s, rows, sets, &p);
  // grid: rows x chunks x head sets
  p.ok = fits && rows * sets * 2 * kMaxTileChunks < 0x7fffffffLL && sets <= 65535;
  return p;
}

TilePlan make_tile_logits_plan(const DecodeShape& s) {
  DecodeShape e = s;
  e.v_axis = CQ_AXIS_TOKEN;
  e.v_group = e.d;
  return make_tile_plan(e);
}

namespace {

// the arguments that both passes read, and the logits launch
hipError_t start_logits(TileArgs& a, const DecodeShape& s, const TilePlan& plan, const void* q,
                        const cq_qtensor_t& k, const void* k_text, const int32_t* n_text_dev,
                        float softmax_scale, float* logits, float* minmax, hipStream_t stream) {
  if (!plan.ok) return hipErrorInvalidValue;
  a.q = static_cast<const __half*>(q);
  a.k_codes = k.codes; a.k_scale = k.scale; a.k_min = k.min;
  a.k_text = static_cast<const __half*>(k_text);
  a.g = s.g; a.sets = ceil_div(s.g, kHeads); a.n_vis = s.n_vis; a.n_text = s.n_text;
  a.n_text_cap = s.n_text_cap; a.n_text_dev = n_text_dev;
  a.k_group = s.k_group; a.k_block = kKeyBlock; a.k_bpg = ceil_div(s.k_group, kKeyBlock);
  a.ca = plan.ca; a.ct = plan.ct; a.ct_tokens = plan.ct_tokens;
  if (s.n_vis > 0) {
    a.k_groups = s.n_vis / s.k_group;
    const int blocks = a.k_groups * a.k_bpg;
    a.ca_base = blocks / a.ca; a.ca_rem = blocks % a.ca;
  }
  a.ws_logits = logits;
  a.ws_minmax = minmax;
  a.softmax_scale = softmax_scale;
  const TileKernel kern = s.d == 64 ? logits_kernel<64>(s.bits)
                          : s.d == 128 ? logits_kernel<128>(s.bits) : logits_kernel<256>(s.bits);
  if (!kern) return hipErrorInvalidValue;
  kern<<<dim3((unsigned)(s.B * s.Hkv), (unsigned)(a.ct + a.ca + a.x_ct), (unsigned)a.sets), dim3(kThreads), 0, stream>>>(a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_tile_logits(const DecodeShape& s, const TilePlan& plan, const void* q,
                              const cq_qtensor_t& k, const void* k_text, float softmax_scale,
                              float* logits, float* minmax, const TilePlan& x_plan, const void* x_keys,
                              int x_tokens, float* x_logits, float* x_minmax, hipStream_t stream) {
  TileArgs a{};
  a.x_keys = static_cast<const __half*>(x_keys);
  a.x_tokens = x_tokens; a.x_ct = x_plan.ct; a.x_ct_tokens = x_plan.ct_tokens;
  a.x_logits = x_logits; a.x_minmax = x_minmax;
  return start_logits(a, s, plan, q, k, k_text, nullptr, softmax_scale, logits, minmax, stream);
}

namespace {

hipError_t launch_tile_rows(const DecodeShape& s, const TilePlan& plan, const void* q, const cq_qtensor_t& k,
                            const cq_qtensor_t& v, const void* k_text, const void* v_text, const int32_t* n_text_dev,
                            const Calib& calib, float softmax_scale, void* out, float* workspace, hipStream_t stream) {
  TileArgs a{};
  const bool vch = s.v_axis == CQ_AXIS_CHANNEL;
  a.q = static_cast<const __half*>(q);
  a.k_codes = k.codes; a.k_scale = k.scale; a.k_min = k.min;
  a.v_codes = v.codes; a.v_scale = v.scale; a.v_min = v.min;
  a.k_text = static_cast<const __half*>(k_text);
  a.v_text = static_cast<const __half*>(v_text);
  a.out = static_cast<__half*>(out);
  a.g = s.g; a.sets = ceil_div(s.g, kHeads); a.n_vis = s.n_vis; a.n_text = s.n_text;
  a.n_text_cap = s.n_text_cap; a.n_text_dev = n_text_dev;
  a.cb = plan.row_cb; a.ct = plan.row_ct; a.ct_tokens = plan.ct_tokens;
  int tokens = plan.ct > 0 ? plan.ct_tokens : 0;               // of the longest chunk
  if (s.n_vis > 0) {
    const int units = ceil_div(s.n_vis, kUnit), per_chunk = ceil_div(units, a.cb);
    a.cb_base = units / a.cb; a.cb_rem = units % a.cb;
    // a block of keys per wave where a chunk is short
    a.k_block = per_chunk >= kWaves ? kKeyBlock : per_chunk > 1 ? kKeyBlock / 2 : kKeyBlock / 4;
    a.k_group = s.k_group; a.k_bpg = ceil_div(s.k_group, a.k_block); a.k_groups = s.n_vis / s.k_group;
    a.k_blocks = a.k_groups * a.k_bpg;
    a.k_bpu = s.k_group < kUnit && s.k_group != s.n_vis ? kUnit / s.k_group * a.k_bpg : kUnit / a.k_block;
    a.v_group = vch ? s.v_group : s.n_vis; a.v_tpg = ceil_div(a.v_group, kValTile); a.v_groups = s.n_vis / a.v_group;
    a.v_tiles = a.v_groups * a.v_tpg;
    a.v_tpu = a.v_group < kUnit && a.v_group != s.n_vis ? kUnit / a.v_group * a.v_tpg : kUnit / kValTile;
    if (per_chunk * kUnit > tokens) tokens = per_chunk * kUnit;
  }
  a.l_stride = (tokens + 63) / 64 * 64 + 16;                   // four heads' rows of 16 lanes on different banks
  a.softmax_scale = softmax_scale;
  a.calib_mode = calib.mode; a.tau1 = calib.tau1; a.tau2 = calib.tau2;
  a.gamma = calib.gamma; a.delta = calib.delta;
  a.ws_words = reinterpret_cast<u64*>(workspace);
  a.ws_tags = reinterpret_cast<u64*>(workspace + plan.row_tags_floats);
  a.ws_partial = workspace + plan.row_partial_floats;
  a.tag = meeting_tag();
  a.patience = plan.patience;
  const unsigned slots = (unsigned)(a.cb + a.ct);
  a.slots_magic = slots == 1 ? 0u : (unsigned)((1ull << 32) / slots + 1);
  const TileKernel kern = s.d == 64 ? row_kernel<64>(s.bits, vch)
                          : s.d == 128 ? row_kernel<128>(s.bits, vch) : row_kernel<256>(s.bits, vch);
  if (!kern) return hipErrorInvalidValue;
  const size_t blocks = (size_t)s.B * s.Hkv * a.sets * slots;
  kern<<<dim3((unsigned)blocks), dim3(kThreads), (size_t)kHeads * a.l_stride * sizeof(float), stream>>>(a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_decode_tile(const DecodeShape& s, const TilePlan& plan, const void* q,
                              const cq_qtensor_t& k, const cq_qtensor_t& v, const void* k_text,
                              const void* v_text, const int32_t* n_text_dev, const Calib& calib,
                              float softmax_scale, void* out, float* workspace, hipStream_t stream) {
  if (plan.ok && (calib.mode == CQ_CALIB_DYNAMIC ? plan.one_launch : plan.one_launch_free))
    return launch_tile_rows(s, plan, q, k, v, k_text, v_text, n_text_dev, calib, softmax_scale, out, workspace, stream);
  TileArgs a{};
  a.ws_count = reinterpret_cast<int*>(workspace + plan.ws_count_floats);
  a.out = static_cast<__half*>(out);
  hipError_t e = start_logits(a, s, plan, q, k, k_text, n_text_dev, softmax_scale, workspace,
                              workspace + plan.ws_minmax_floats, stream);
  if (e != hipSuccess) return e;
  a.v_codes = v.codes; a.v_scale = v.scale; a.v_min = v.min;
  a.v_text = static_cast<const __half*>(v_text);
  const bool vch = s.v_axis == CQ_AXIS_CHANNEL;
  a.v_group = vch ? s.v_group : s.n_vis; a.v_tpg = ceil_div(a.v_group, kValTile);
  a.cb = plan.cb;
  if (s.n_vis > 0) {
    a.v_groups = s.n_vis / a.v_group;
    const int tiles = a.v_groups * a.v_tpg;
    a.cb_base = tiles / a.cb; a.cb_rem = tiles % a.cb;
  }
  a.ws_partial = workspace + plan.ws_partial_floats;
  a.calib_mode = calib.mode; a.tau1 = calib.tau1; a.tau2 = calib.tau2;
  a.gamma = calib.gamma; a.delta = calib.delta;
  const TileKernel kern = s.d == 64 ? values_kernel<64>(s.bits, vch)
                          : s.d == 128 ? values_kernel<128>(s.bits, vch) : values_kernel<256>(s.bits, vch);
  if (!kern) return hipErrorInvalidValue;
  kern<<<dim3((unsigned)(s.B * s.Hkv), (unsigned)(a.ct + a.cb), (unsigned)a.sets), dim3(kThreads), 0, stream>>>(a);
  return hipGetLastError();
}

}  // namespace cq
