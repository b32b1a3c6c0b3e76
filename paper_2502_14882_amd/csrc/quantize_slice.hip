// Channel-wise groups that a workgroup's registers hold (gfx950): any head_dim, b in {1, 2, 4, 8}, groups of 129 to a
// few thousand tokens - one pair per channel over the whole sequence, Sec. 3.1 as printed, on an image or two - where
// that is faster (quantize_slice_supported).
//
// The tile kernels of quantize_tile.h read such a group twice: once for its extrema, once for its codes, with launches
// in between.  Here a workgroup owns 32 or 64 channels of a group, all its tokens: it reads them once, 64 or 128
// bytes per token, keeps them in registers, takes extrema and thresholds in LDS, and forms the codes (steps 1 to
// 3 of quantize_tile.h, with the same arithmetic: the same bits).  Nothing crosses workgroups, one launch does
// both tensors, and no output buffer holds intermediate results.
//
// Layout.  A thread holds 8 channels (16 bytes) of every kTokens-th token; 4 or 8 lanes hold a token's piece.  The
// slices of a group lie in the same cache lines, both where they read and where they write their codes, so they get
// block indices 8 apart: the same XCD, at the same time, and its L2 puts the lines together.
//
// Bound: what a CU reads (a workgroup's loads are all out before its arithmetic begins, 16 waves to a CU) and
// vector issue, one behind the other unless a workgroup takes several blocks (slice_kernel).  Keys and values, tile
// kernels / here, us, call after call on the same tensors: 64 rows x 3003 tokens, 2 bits 42.9 / 22.3 (here 29.6 where the tensors
// change from call to call); 256 x 2000 101 / 57.6; 8 x 1000, 1 bit 8.8 / 3.8; 512 x 300 34.5 / 15.5; 64 x 3003 of 64 channels, 2 bits
// 25.6 / 13.5; at the longest, 4096 tokens, 64 x, 1 bit 49.1 / 25.2, 2 bits 55.1 / 29.9, 256 x, 2 bits 205 / 158.
#include <hip/hip_fp16.h>

#include "cq_internal.h"
#include "quantize_tile.h"

namespace cq {
namespace {

struct SliceArgs {
  const __half* x;
  uint32_t* codes;
  float* scale;
  uint16_t* minv;
};

// grid: ((group / 8) * slices + slice) * 8 + group % 8, first the one tensor's groups, then the other's
// ROUNDS: a workgroup has a CU to itself and takes every gridDim.x-th block, one behind the other; as soon as a piece of x
// has become codes, the same piece of the next block is asked for.
template <int BITS, int LANES, int THREADS, int P, bool ROUNDS>
__global__ void __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(BITS <= 2 || P <= 12 ? 4 : 1)))
quantize_slice_kernel(const SliceArgs first, const SliceArgs second, int n_first, int n_groups, int tokens, int d,
                      int log_slices, int n_blocks) {
  constexpr int L = (1 << BITS) - 1, kTokens = THREADS / LANES, kSlice = 8 * LANES, kWavesQ = THREADS / 64;
  constexpr bool kWide = BITS > 2;
  __shared__ __align__(16) _Float16 s_part[2][kWavesQ][kSlice];
  __shared__ __align__(16) _Float16 s_thr[kWide ? 1 : L][kSlice];
  __shared__ __align__(16) double s_rinv[kWide ? kSlice : 1];
  __shared__ __align__(16) _Float16 s_alpha[kSlice];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, oct = lane & (LANES - 1);
  int t_lane = tid / LANES;
  struct Piece { bool one; int group, c0; };
  auto piece_of = [&](int block) {
    const int slot = block >> 3, group = (slot >> log_slices) * 8 + (block & 7);
    return Piece{group < n_first, group < n_first ? group : group - n_first, (slot & ((1 << log_slices) - 1)) * kSlice};
  };
  auto exists = [&](int block) {                // the blocks are whole eights of groups
    return block < n_blocks && (block >> 3 >> log_slices) * 8 + (block & 7) < n_groups;
  };
  auto source = [&](const Piece& p) {
    return reinterpret_cast<const char*>((p.one ? first.x : second.x) + (size_t)p.group * tokens * d + p.c0);
  };
  auto load = [&](const char* src, int i) {     // past the end: the last token, which changes no extremum
    const int t0 = min(i * kTokens, tokens - 1);
    return *reinterpret_cast<const v8h*>(src + (size_t)t0 * (unsigned)(2 * d) +
                                         ((unsigned)min(t_lane, tokens - 1 - t0) * (unsigned)(2 * d) + 16u * oct));
  };
  int block = (int)blockIdx.x;
  if (!exists(block)) return;
  Piece piece = piece_of(block);
  v8h x[P];                                     // read exactly once
  {
    const char* src = source(piece);
#pragma unroll
    for (int i = 0; i < P; ++i) x[i] = load(src, i);
  }
  for (;;) {
    // (offsets of loads and stores are made anew in every round: kept from round to round they spill)
    if constexpr (ROUNDS) asm volatile("" : "+v"(t_lane));
    const bool one = piece.one;
    const int group = piece.group, c0 = piece.c0;
    const size_t tok0 = (size_t)group * tokens;
    bool more = false;
    if constexpr (ROUNDS) {
      block += (int)gridDim.x;
      more = exists(block);
      if (more) piece = piece_of(block);
    }
    const char* next = source(piece);
    // ---- 1. extrema of the slice's channels
    v8h mn = x[0], mx = x[0];
#pragma unroll
    for (int i = 1; i < P; ++i) {
      mn = __builtin_elementwise_min(mn, x[i]);
      mx = __builtin_elementwise_max(mx, x[i]);
    }
    store_extrema<LANES>(mn, mx, lane, s_part[0][wave], s_part[1][wave]);
    __syncthreads();
    // ---- 2. stored parameters; a thread per (threshold, channel)
    constexpr int kEach = kWide ? 1 : L;
    if (tid < kEach * kSlice) {
      const int c = tid & (kSlice - 1), k = tid / kSlice + 1;
      _Float16 lo = s_part[0][0][c], hi = s_part[1][0][c];
#pragma unroll
      for (int w = 1; w < kWavesQ; ++w) {
        lo = (_Float16)fminf((float)lo, (float)s_part[0][w][c]);
        hi = (_Float16)fmaxf((float)hi, (float)s_part[1][w][c]);
      }
      const uint16_t mbits = canonical_zero(__builtin_bit_cast(uint16_t, lo));
      const double alpha = h_to_double(mbits);
      const double range = ((double)(float)hi - alpha) + 0.0;
      if (k == 1) {
        const size_t meta = (size_t)group * d + c0 + c;
        (one ? first.scale : second.scale)[meta] = (float)(range / (double)L);
        (one ? first.minv : second.minv)[meta] = mbits;
      }
      if constexpr (kWide) {
        s_alpha[c] = __builtin_bit_cast(_Float16, mbits);
        s_rinv[c] = range > 0.0 ? (double)L / range : 0.0;
      } else {
        s_thr[k - 1][c] = __builtin_bit_cast(_Float16, threshold_bits(alpha, range, k, L));
      }
    }
    __syncthreads();
    // ---- 3. codes: BITS words per token and slice
    const int words = d * BITS / 32;
    uint32_t* dst = (one ? first.codes : second.codes) + tok0 * words + c0 / 32 * BITS;
    if constexpr (kWide) {
      double al[8], ri[8];
      float al32[8], ri32[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        al32[j] = (float)s_alpha[8 * oct + j];
        al[j] = (double)al32[j];
        ri[j] = s_rinv[8 * oct + j];
        ri32[j] = (float)ri[j];
      }
      static_assert(!ROUNDS, "one and two bits: with wider codes the loop spills");
#pragma unroll
      for (int i = 0; i < P; ++i) {
        uint32_t* to = dst + (size_t)(i * kTokens) * (unsigned)words;
        const unsigned at = (unsigned)t_lane * (unsigned)words;
        uint32_t w0, w1;
        octet_words<BITS>(x[i], al, ri, al32, ri32, w0, w1);
        if (t_lane < tokens - i * kTokens) {
          if constexpr (BITS == 4) to[at + oct] = w0;
          else *reinterpret_cast<v2u*>(to + (at + 2 * oct)) = (v2u){w0, w1};
        }
      }
    } else {
      v8h thr[L];
#pragma unroll
      for (int k = 0; k < L; ++k) thr[k] = *reinterpret_cast<const v8h*>(&s_thr[k][8 * oct]);
      auto put = [&](int i) {
        uint32_t* to = dst + (size_t)(i * kTokens) * (unsigned)words;
        const unsigned at = (unsigned)t_lane * (unsigned)words;
        uint32_t bits = octet_codes<BITS>(x[i], thr);
        if constexpr (BITS == 1) {
          bits <<= 24 - 8 * (oct & 3);
          bits |= other_lane<0xB1>(bits);
          bits |= other_lane<0x4E>(bits);
          if ((oct & 3) == 0 && t_lane < tokens - i * kTokens) to[at + (oct >> 2)] = bits;
        } else {
          bits <<= 16 - 16 * (oct & 1);
          bits |= other_lane<0xB1>(bits);
          if ((oct & 1) == 0 && t_lane < tokens - i * kTokens) to[at + (oct >> 1)] = bits;
        }
      };
      if (more) {
#pragma unroll
        for (int i = 0; i < P; ++i) {
          put(i);
          x[i] = load(next, i);
        }
      } else {
#pragma unroll
        for (int i = 0; i < P; ++i) put(i);
      }
    }
    if (!more) return;
  }
}

using SliceKernel = void (*)(const SliceArgs, const SliceArgs, int, int, int, int, int, int);
// Whole lines per token (8 lanes) where the group is short; else half of one, with which more workgroups share a CU
// (us, one-bit keys and values, 8 / 4 lanes: 512 rows x 300 tokens 17.1 / 27.3, 8 x 1000 5.7 / 4.5, 256 x 2000 with two
// bits 86.6 / 70.6; 8 bits, 256 x 1500 83.5 / 95.1).  Beyond 2048 tokens 1024 threads; 24 registers of data per
// thread instead are slower (64 x 3003 41.6 / 37.8).  (These are from before the codes took half the instructions; the kernels
// chosen have since become faster by a tenth to a fifth, the others were not measured again.)
// Where such a workgroup leaves no room for another (1024 threads) and there are more of them than CUs, one to a CU takes
// its blocks in rounds: us, a workgroup per block / in rounds: 2 bits 64 x 3003 31.5 / 29.6, 256 x 3003 122 / 113, 96 x 2049
// 36.0 / 32.0, 64 channels 128 x 3003 32.1 / 28.8; 1 bit 64 x 3003 24.8 / 24.5, 128 x 4000 67.0 / 63.3.  Not with 256 channels, eight
// slices to a line of tokens: 160 x 2500 127 / 138, 160 x 4000, 1 bit 161 / 178.
template <int BITS>
SliceKernel slice_kernel(int tokens, int d, long long blocks_of_4_lanes, int* threads, int* lanes, bool* rounds) {
  *lanes = 8;
  *threads = 512;
  *rounds = false;
  if (tokens <= 512) return quantize_slice_kernel<BITS, 8, 512, 8, false>;
  *lanes = 4;
  if (tokens <= 1024) return quantize_slice_kernel<BITS, 4, 512, 8, false>;
  if constexpr (BITS <= 2) {
    if (tokens <= 2048) return quantize_slice_kernel<BITS, 4, 512, 16, false>;
    *threads = 1024;
    if (tokens > 4096) return nullptr;
    *rounds = d <= 128 && blocks_of_4_lanes > device_cu_count();
    if (tokens <= 3072) return *rounds ? quantize_slice_kernel<BITS, 4, 1024, 12, true> : quantize_slice_kernel<BITS, 4, 1024, 12, false>;
    return *rounds ? quantize_slice_kernel<BITS, 4, 1024, 16, true> : quantize_slice_kernel<BITS, 4, 1024, 16, false>;
  } else {
    *threads = 1024;
    *lanes = 8;
    if (tokens <= 1536) return quantize_slice_kernel<BITS, 8, 1024, 12, false>;
    *lanes = 4;
    return tokens <= 3072 ? quantize_slice_kernel<BITS, 4, 1024, 12, false> : nullptr;
  }
}

}  // namespace

// A workgroup's own time grows with the tokens it owns and the width of the codes, so long groups take the tile kernels'
// many workgroups unless there are enough of them, and beyond 3072 tokens 4- and 8-bit codes always do (their registers
// spilled there: 8 bits, 4000 tokens, 128 channels in all 14.7 / 21.9, 8192 74.6 / 76.0).  us, keys and values whole, tile
// kernels / here: 4 bits 1500 tokens, 64 channels in all 9.3 / 10.3, 128 11.4 / 10.6; 3000 tokens 1024 15.0 / 11.9; 8 bits 1500
// tokens 64 10.5 / 10.8, 128 13.8 / 12.2; 3000 tokens 1024 17.8 / 14.2.  One bit always wins.  The lines for the longest groups
// were drawn when a block here took half as long again (2 bits 4000 tokens 128 channels 13.6 / 15.5, 4 bits 3000 13.2 / 14.6); now
// they keep calls from the faster kernel: 2 bits 4000 tokens 128 and 256 channels 11.3 / 9.4, 3003 tokens 64 channels 9.3 /
// 7.7, 4 bits 3000 tokens 128 and 256 channels 11.9 / 11.3, 12.4 / 11.3, 8 bits 128 13.2 / 12.8.
bool quantize_slice_supported(size_t n_tokens, int d, int bits, int axis, int group) {
  if (axis != CQ_AXIS_CHANNEL || group <= kTile || group > (bits <= 2 ? 4096 : 3072)) return false;
  if (d != 64 && d != 128 && d != 256) return false;
  const size_t channels = n_tokens / group * d;                // of all groups
  const size_t least = bits == 1 ? 0 : bits == 2 ? (group <= 2048 ? 0 : group <= 3072 ? 128 : 512) : group <= 1024 ? 0
                       : group <= 1536 ? 128 : 512;
  if (channels < least) return false;
  // two tensors of whole eights of groups in one grid of at most 2^32 - 1 threads
  return (n_tokens / group * 2 + 8) * (d / 32) <= 0xffffffffu / 1024;
}

hipError_t launch_quantize_slices(const QuantizeJob* jobs, int n_jobs, size_t n_tokens, int d, int bits, hipStream_t stream) {
  const int tokens = jobs[0].group, n = (int)(n_tokens / tokens);
  const int groups = n * n_jobs, log_slices_4 = d == 64 ? 1 : d == 128 ? 2 : 3;
  const unsigned eights = (unsigned)((groups + 7) / 8 * 8);
  const long long blocks_4 = (long long)eights << log_slices_4;
  int threads = 0, lanes = 0;
  bool rounds = false;
  const auto pick = bits == 1 ? slice_kernel<1> : bits == 2 ? slice_kernel<2> : bits == 4 ? slice_kernel<4> : slice_kernel<8>;
  const SliceKernel kern = pick(tokens, d, blocks_4, &threads, &lanes, &rounds);
  if (!kern) return hipErrorInvalidValue;
  auto args = [](const QuantizeJob& j) {
    return SliceArgs{static_cast<const __half*>(j.x_f16), j.out.codes, j.out.scale, j.out.min};
  };
  const int log_slices = log_slices_4 - (lanes == 8 ? 1 : 0);
  const unsigned blocks = eights << log_slices;
  const unsigned grid = rounds ? (unsigned)device_cu_count() & ~7u : blocks;      // whole eights: a block stays on its XCD
  kern<<<dim3(grid), dim3((unsigned)threads), 0, stream>>>(args(jobs[0]), args(jobs[n_jobs - 1]), n, groups, tokens, d,
                                                           log_slices, (int)blocks);
  return hipGetLastError();
}

}  // namespace cq
