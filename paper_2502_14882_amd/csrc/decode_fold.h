// Folds over the wave for floats and doubles alike, on the vector unit (DPP moves and lane swaps).
// Internal to libcq; used by decode_tile.hip and calib_search.hip.
#ifndef CQ_DECODE_FOLD_H_
#define CQ_DECODE_FOLD_H_

#include "decode_device.h"

namespace cq {
namespace {

// The same lane moves for doubles, half by half.
template <int CTRL>
__device__ inline double dpp_f64(double v) {
  const v2i x = __builtin_bit_cast(v2i, v);
  const v2i r = {__builtin_amdgcn_update_dpp(x[0], x[0], CTRL, 0xF, 0xF, true),
                 __builtin_amdgcn_update_dpp(x[1], x[1], CTRL, 0xF, 0xF, true)};
  return __builtin_bit_cast(double, r);
}
template <int CTRL> __device__ inline float dpp_move(float v) { return dpp_f32<CTRL>(v); }
template <int CTRL> __device__ inline double dpp_move(double v) { return dpp_f64<CTRL>(v); }
// a + (a of the other half of the wave) in lanes 0-31, the same of b in lanes 32-63: a paired swap of
// two values and one add halve both
__device__ inline float fold_halves(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b), false, false);
  return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}
__device__ inline double fold_halves(double a, double b) {
  const v2u x = __builtin_bit_cast(v2u, a), y = __builtin_bit_cast(v2u, b);
  const auto lo = __builtin_amdgcn_permlane32_swap(x[0], y[0], false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(x[1], y[1], false, false);
  return __builtin_bit_cast(double, (v2u){lo[0], hi[0]}) + __builtin_bit_cast(double, (v2u){lo[1], hi[1]});
}
// the same over neighbouring rows of 16 lanes
__device__ inline float fold_rows(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b), false, false);
  return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}
__device__ inline double fold_rows(double a, double b) {
  const v2u x = __builtin_bit_cast(v2u, a), y = __builtin_bit_cast(v2u, b);
  const auto lo = __builtin_amdgcn_permlane16_swap(x[0], y[0], false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(x[1], y[1], false, false);
  return __builtin_bit_cast(double, (v2u){lo[0], hi[0]}) + __builtin_bit_cast(double, (v2u){lo[1], hi[1]});
}

// the larger of the two halves' values, and of neighbouring rows', in every lane
template <int CTRL>
__device__ inline int dpp_i32(int v) { return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xF, 0xF, true); }
__device__ inline int max_halves(int v) {
  const auto r = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
  return max((int)r[0], (int)r[1]);
}
__device__ inline int max_rows(int v) {
  const auto r = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
  return max((int)r[0], (int)r[1]);
}

// Sum over the wave of the four heads' parts, head kb = lane / 16 in every lane of row kb.  A
// transposing butterfly leaves lane (.., b1, b0) with head 2*b0 + b1 after two steps, the remaining
// steps add lanes that hold the same head.  Every lane of a row then holds the row's sum for head
// bitrev2(lane & 3); what is wanted is the sum over the four rows, head kb in row kb: the four heads
// side by side (quad broadcasts), then a transposing fold over the rows with paired lane swaps.  (The
// fold inside group_bias of decode_device.h, for either type.)
template <typename T>
__device__ inline T head_sums(const T (&part)[kHeads], int lane) {
  const bool b0 = lane & 1, b1 = lane & 2;
  T u0 = b0 ? part[2] : part[0], u1 = b0 ? part[3] : part[1];
  const T g0 = b0 ? part[0] : part[2], g1 = b0 ? part[1] : part[3];
  u0 += dpp_move<0xB1>(g0);                // quad_perm 1,0,3,2: lane ^ 1
  u1 += dpp_move<0xB1>(g1);
  T r = b1 ? u1 : u0;
  const T g2 = b1 ? u0 : u1;
  r += dpp_move<0x4E>(g2);                 // quad_perm 2,3,0,1: lane ^ 2
  r += dpp_move<0x124>(r);                 // row_ror 4
  r += dpp_move<0x128>(r);                 // row_ror 8
  const T h0 = dpp_move<0x00>(r), h1 = dpp_move<0xAA>(r);     // quad lanes 0 and 2
  const T h2 = dpp_move<0x55>(r), h3 = dpp_move<0xFF>(r);     // quad lanes 1 and 3
  // heads 0 | 2 and 1 | 3 in the halves, then rows 0..3: heads 0, 1, 2, 3
  return fold_rows(fold_halves(h0, h2), fold_halves(h1, h3));
}

// ---- operands in fixed point that keep fp32's bits
// The four signed base-256 digits of a * b rounded to the nearest integer (|a b| < 2^30), as the four
// bytes of the result.  Added to 1.5 * 2^52 a double shows the integer in its low word.
__device__ inline int rounded_digits(float a, double b) {
  const double t = fma((double)a, b, 6755399441055744.0 + 8421504.0);
  return __builtin_bit_cast(v2i, t)[0] ^ 0x00808080;
}

// a * b + the bias of the four signed base-256 digits: as an integer ^ 0x00808080 its bytes are the digits.
// Above 2^23 the fma rounds to nearest integers, and fp32 has no more below 2^24.
__device__ inline float digits_bias(float a, float b) { return fmaf(a, b, 8421504.f); }

// Fixed-point scales of the four heads, powers of two from 2^-90 to 2^90, as the bits of floats.
struct Scales {
  static constexpr int kOne = 127 << 23;
  int up[kHeads];                                              // wave-uniform
  __device__ explicit Scales(int exponent) {
#pragma unroll
    for (int h = 0; h < kHeads; ++h) up[h] = (exponent + 127) << 23;
  }
  __device__ float of(int h) const { return __builtin_bit_cast(float, up[h]); }
  __device__ float inverse(int kb) const {                     // of head kb
    const int a = kb & 1 ? up[1] : up[0], b = kb & 1 ? up[3] : up[2];
    return __builtin_bit_cast(float, 2 * kOne - (kb & 2 ? b : a));
  }
  // Lowered until w * scale < 2^26 for the heads' w >= 0 of all lanes.  The maxima by a transposing
  // butterfly, as in head_sums: lane l of a row ends up with head bitrev2(l & 3).  Floats that are not
  // negative order like their bits, and integer maxima need no second instruction for NaNs.
  __device__ void lower(const float (&w)[kHeads], int lane) {
    const bool b0 = lane & 1, b1 = lane & 2;
    int i[kHeads];
#pragma unroll
    for (int h = 0; h < kHeads; ++h) i[h] = __builtin_bit_cast(int, w[h]);
    const int u0 = max(b0 ? i[2] : i[0], dpp_i32<0xB1>(b0 ? i[0] : i[2]));
    const int u1 = max(b0 ? i[3] : i[1], dpp_i32<0xB1>(b0 ? i[1] : i[3]));
    int r = max(b1 ? u1 : u0, dpp_i32<0x4E>(b1 ? u0 : u1));
    r = max(r, dpp_i32<0x124>(r));
    r = max_rows(max_halves(max(r, dpp_i32<0x128>(r))));
    // r < 2^(e - 126) for its exponent field e: the scale 2^(26 - (e - 126)), its field 279 - e
    const int fits = min(max(279 - (r >> 23), 127 - 90), 127 + 90) << 23;
    constexpr int kLane[kHeads] = {0, 2, 1, 3};
#pragma unroll
    for (int h = 0; h < kHeads; ++h) up[h] = min(up[h], __builtin_amdgcn_readlane(fits, kLane[h]));
  }
};

}  // namespace
}  // namespace cq

#endif  // CQ_DECODE_FOLD_H_
