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
// merges, in the order of the chunks, so the result does not depend on who that is.  It also clears the words
// and the count, which nobody reads any more: a recorded launch finds them clear when it is replayed with the
// same tag.
#ifndef CQ_DECODE_MEET_H_
#define CQ_DECODE_MEET_H_

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
// The workgroups counted before this one.  seen: what count_open returned.  Memory that held something
// else takes a second exchange; whoever's succeeds, the word then counts for the call.
__device__ inline int count_in(u64* count, u64 tag, u64 seen) {
  if (seen != 0 && (seen & ~(u64)0xff) != tag)
    atomicCAS(count, seen, tag);
  return (int)(__hip_atomic_fetch_add(count, (u64)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 0xff);
}

// ---- merge of the partials [heads][n_slots][D + 2] = (m, l, acc[D]) of gh heads; two channels per thread
template <int D, int THREADS>
__device__ inline void merge_partials(const float* partial, int n_slots, int gh, __half* out) {
  constexpr int kPairs = D / 2;
  for (int e = threadIdx.x; e < gh * kPairs; e += THREADS) {
    const int h = e / kPairs, c = 2 * (e % kPairs);
    const float* base = partial + h * (size_t)n_slots * (D + 2);
    // sixteen partials at a time, their loads independent of each other; each batch brings its own
    // reference point (online softmax over batches).  A chunk without tokens has weight 0.
    float M = -FLT_MAX, den = 0.f;
    v2f num = {0.f, 0.f};
    for (int i0 = 0; i0 < n_slots; i0 += 16) {
      v2f ml[16], acc[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const float* p = base + (size_t)min(i0 + u, n_slots - 1) * (D + 2);
        ml[u] = load_device(p);
        acc[u] = load_device(p + 2 + c);
      }
      float Mb = M;
#pragma unroll
      for (int u = 0; u < 16; ++u) Mb = fmaxf(Mb, ml[u][0]);     // a repeated partial changes nothing
      const float keep = __builtin_amdgcn_exp2f((M - Mb) * kLog2e);
      num *= keep;
      den *= keep;
      M = Mb;
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const float w = i0 + u < n_slots ? __builtin_amdgcn_exp2f((ml[u][0] - M) * kLog2e) : 0.f;
        num[0] = fmaf(w, acc[u][0], num[0]);
        num[1] = fmaf(w, acc[u][1], num[1]);
        den = fmaf(w, ml[u][1], den);
      }
    }
    *reinterpret_cast<__half2*>(out + h * D + c) = __floats2half2_rn(num[0] / den, num[1] / den);
  }
}

}  // namespace

// A number that no other call has (64 bits, mixed; the low byte is zero and neither half is).
u64 meeting_tag();

}  // namespace cq

#endif  // CQ_DECODE_MEET_H_
