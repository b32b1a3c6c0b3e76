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

}  // namespace
}  // namespace cq

#endif  // CQ_DECODE_FOLD_H_
