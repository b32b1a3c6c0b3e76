// Rows that several workgroups of ONE launch share (decode_fused.hip, decode_tile.hip): how these
// exchange the extrema of their logits, and how the last one to finish merges the partials of the online
// softmax.  Internal to libcq; inline device code and the tag of a call.
//
// All of it crosses from one XCD's L2 to another's inside a launch: stored and loaded at device scope,
// eight bytes at a time.
//
// Exchange.  A workgroup stores the extrema of its logits as two words that carry a tag of the call and
// check each other: memory that holds anything else - the workspace comes with undefined contents - is not
// taken for them.  A reader looks until all words of its row are there, a BOUNDED number of times: the
// workgroups of a row have neighbouring indices and are started together, but nothing promises that they are
// all resident (other work may hold the compute units), so a reader that has looked in vain forms the
// extrema of the whole row itself.  No workgroup's end depends on another's start.
//
// Merge.  Every workgroup counts itself when its partial has reached memory; the one that counts last
// merges, in the order of the chunks, so the result does not depend on who that is.  It also clears the
// count, and the words where no partials have taken their place, which nobody reads any more: a recorded launch
// finds nothing of its own when it is replayed with the same tag.
#ifndef CQ_DECODE_MEET_H_
#define CQ_DECODE_MEET_H_

#include <type_traits>

#include "decode_device.h"

namespace cq {
namespace {

typedef unsigned long long u64;

// ---- device scope
__device__ inline void store_device(float* p, float a, float b) {
  __hip_atomic_store(reinterpret_cast<u64*>(p), __builtin_bit_cast(u64, (v2f){a, b}), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void store_device(float* p, float a) {
  __hip_atomic_store(p, a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline v2f load_device(const float* p) {
  return __builtin_bit_cast(v2f, __hip_atomic_load(reinterpret_cast<const u64*>(p), __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT));
}

// ---- exchange: words [heads][chunks][2]
__device__ inline void post_extrema(u64* w, float lo, float hi, u64 tag) {
  const unsigned a = __builtin_bit_cast(unsigned, lo), b = __builtin_bit_cast(unsigned, hi);
  const u64 w0 = (u64)((unsigned)tag ^ b) << 32 | a, w1 = (u64)((unsigned)(tag >> 32) ^ a) << 32 | b;
  __hip_atomic_store(w, w0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(w + 1, w1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline bool read_extrema(const u64* w, float* lo, float* hi, u64 tag) {
  const u64 w0 = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const u64 w1 = __hip_atomic_load(w + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const unsigned a = (unsigned)w0, b = (unsigned)w1;
  *lo = __builtin_bit_cast(float, a);
  *hi = __builtin_bit_cast(float, b);
  return (unsigned)(w0 >> 32) == ((unsigned)tag ^ b) && (unsigned)(w1 >> 32) == ((unsigned)(tag >> 32) ^ a);
}

// ---- count: the tag with the number of workgroups so far in its low byte (a tag ends in a zero byte)
// Asked for at the start of a workgroup; clear memory (0) becomes the tag.
__device__ inline u64 count_open(u64* count, u64 tag) {
  return atomicCAS(count, (u64)0, tag);
}
// Whether a workgroup of the call has been counted.
__device__ inline bool any_counted(const u64* count, u64 tag) {
  const u64 c = __hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return __builtin_amdgcn_readfirstlane((int)((c & ~(u64)0xff) == tag && (c & 0xff) != 0)) != 0;
}
// The workgroups counted before this one.  seen: what count_open returned.  Memory that held something
// else takes a second exchange; whoever's succeeds, the word then counts for the call.
__device__ inline int count_in(u64* count, u64 tag, u64 seen) {
  if (seen != 0 && (seen & ~(u64)0xff) != tag)
    atomicCAS(count, seen, tag);
  return (int)(__hip_atomic_fetch_add(count, (u64)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 0xff);
}

// ---- merge of the partials [heads][n_slots][D + 2] = (m, l, acc[D]) of gh <= 4 heads
// A wave takes one head and every kGroups-th slot, its lanes the channels; the (m, l) of up to 64 slots come in
// one load, a lane each.  A chunk without tokens has weight 0.  lds: kGroups * 4 * D floats that nobody reads
// any more.  (One thread per pair of channels over all slots, sixteen at a time whether there are sixteen or not,
// took 1.0 to 1.5 us of a call; this takes 0.5.)
template <int D, int WAVES>
__device__ inline void merge_partials(const float* partial, int n_slots, int gh, __half* out, float* lds, int tid) {
  constexpr int kGroups = WAVES / kHeads, kPer = D / 64;       // channels per lane
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = wave % kHeads, first = wave / kHeads;
  float num[kPer], den = 0.f;
#pragma unroll
  for (int e = 0; e < kPer; ++e) num[e] = 0.f;
  if (h < gh) {
    const float* base = partial + h * (size_t)n_slots * (D + 2);
    float M = -FLT_MAX;
    auto take = [&](auto batch_tag, int s0, int n) {           // n <= 64 slots, BATCH loads in flight
      constexpr int BATCH = decltype(batch_tag)::value;
      const v2f ml = load_device(base + (size_t)(s0 + min(lane, n - 1)) * (D + 2));
      float acc[BATCH][kPer];
      auto load = [&](int i0) {
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
          const float* p = base + (size_t)(s0 + min(i0 + u * kGroups, n - 1)) * (D + 2) + 2 + kPer * lane;
          if constexpr (kPer == 1) {
            acc[u][0] = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          } else {
#pragma unroll
            for (int e = 0; e < kPer; e += 2) {
              const v2f t = load_device(p + e);
              acc[u][e] = t[0];
              acc[u][e + 1] = t[1];
            }
          }
        }
      };
      load(first);                                             // before anything is done with (m, l)
      // (any slot may be empty, with -FLT_MAX for its m: nothing is formed by differences to a certain one's)
      const float Mb = fmaxf(M, wave_max(ml[0]));
      const float keep = __builtin_amdgcn_exp2f((M - Mb) * kLog2e);
      M = Mb;
      const float w = lane < n ? __builtin_amdgcn_exp2f((ml[0] - M) * kLog2e) : 0.f;
      den = fmaf(den, keep, wave_sum(w * ml[1]));
#pragma unroll
      for (int e = 0; e < kPer; ++e) num[e] *= keep;
      for (int i0 = first;;) {
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
          const int i = i0 + u * kGroups;
          const float wi = i < n ? lane_value(w, i) : 0.f;
#pragma unroll
          for (int e = 0; e < kPer; ++e) num[e] = fmaf(wi, acc[u][e], num[e]);
        }
        i0 += BATCH * kGroups;
        if (i0 >= n) break;
        load(i0);
      }
    };
    if (n_slots <= 4 * kGroups) take(std::integral_constant<int, 4>{}, 0, n_slots);
    else for (int s0 = 0; s0 < n_slots; s0 += 64) take(std::integral_constant<int, 12>{}, s0, min(64, n_slots - s0));
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      if constexpr (kGroups > 1) lds[(first * kHeads + h) * D + kPer * lane + e] = num[e] / den;
      else out[h * D + kPer * lane + e] = __float2half_rn(num[e] / den);
    }
  }
  if constexpr (kGroups > 1) {
    __syncthreads();
    for (int e = tid; e < gh * D; e += WAVES * 64) {
      float sum = 0.f;
#pragma unroll
      for (int f = 0; f < kGroups; ++f) sum += lds[f * kHeads * D + e];
      out[e] = __float2half_rn(sum);
    }
  }
}

}  // namespace

// A number that no other call has (64 bits, mixed; the low byte is zero and neither half is).
u64 meeting_tag();

}  // namespace cq

#endif  // CQ_DECODE_MEET_H_
