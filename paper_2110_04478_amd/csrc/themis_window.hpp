// Windows of a batch: their scenarios in turns of 16 that take about the same time, for
// kernels with four lanes per scenario (themis_quad.hpp).
#pragma once

#include "themis_device.hpp"

namespace themis {

// Scenarios of a window of the batch in turns of 16, the longest first: a turn takes as
// long as its longest, so scenarios of about the same length go together (100,003 ragged
// scenarios of any NPU counts, planner and both simulation kernels: 16 out of 64 neighbours
// 1,095 us, out of 512 656).  Every workgroup that takes turns of a window finds the order
// by itself, from the inputs alone, so nothing is passed between them: lengths in 64
// buckets, inside of a bucket as they come (33 buckets: 624 us of the above, now 615).
constexpr uint32_t kWindow = 512u, kWindowGroups = kWindow / kBlock, kWindowTurns = kWindow / 16u;
struct QuadWindow {
  uint32_t rank[kWindowGroups];   // of the scenarios of the lane, one in each 64 (all-ones: not among them)
  uint32_t total;
  // lengths[g]: that of scenario 64 * g + lane of the window, 0: not among them; most: the
  // largest there can be (33 to 64 of the buckets are in use, all of them where it is a power
  // of two).  All lanes; lds: 1,056 bytes.
  __device__ __forceinline__ QuadWindow(uint32_t most, void* lds, const uint32_t (&lengths)[kWindowGroups]) {
    uint16_t* const count = (uint16_t*)lds;   // of the scenarios of each 64 in each bucket, then how many come before
    const uint32_t lane = threadIdx.x & 63u, bits = 32u - (uint32_t)__clz((int)((most - 1u) | 1u));
    const uint32_t shift = bits > 6u ? bits - 6u : 0u;
    __syncthreads();
#pragma unroll
    for (uint32_t g = 0; g < kWindowGroups; ++g) count[64u * g + lane] = 0u;
    __syncthreads();
    uint32_t bucket[kWindowGroups];
#pragma unroll
    for (uint32_t g = 0; g < kWindowGroups; ++g) {
      const bool member = lengths[g] != 0u;
      bucket[g] = 63u - min(lengths[g] >> shift, 63u);
      uint64_t same = __builtin_amdgcn_ballot_w64(member);
#pragma unroll
      for (uint32_t j = 0; j < 6u; ++j) {
        const bool one = ((bucket[g] >> j) & 1u) != 0u;
        const uint64_t ones = __builtin_amdgcn_ballot_w64(one);
        same &= one ? ones : ~ones;
      }
      const uint32_t before = __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
      rank[g] = member ? before : ~0u;
      if (member && before == 0u) count[64u * g + bucket[g]] = (uint16_t)__builtin_popcountll(same);
    }
    __syncthreads();
    uint32_t mine[kWindowGroups], all = 0u;   // (of bucket `lane`)
#pragma unroll
    for (uint32_t g = 0; g < kWindowGroups; ++g) mine[g] = count[64u * g + lane];
#pragma unroll
    for (uint32_t g = 0; g < kWindowGroups; ++g) all += mine[g];
    uint32_t upto = all;
    for (uint32_t off = 1u; off < 64u; off <<= 1) {
      const uint32_t below = (uint32_t)__shfl_up((int)upto, off);
      upto += lane >= off ? below : 0u;
    }
    total = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
    uint32_t at = upto - all;
#pragma unroll
    for (uint32_t g = 0; g < kWindowGroups; ++g) {
      count[64u * g + lane] = (uint16_t)at;
      at += mine[g];
    }
    __syncthreads();
#pragma unroll
    for (uint32_t g = 0; g < kWindowGroups; ++g)
      rank[g] = rank[g] != ~0u ? count[64u * g + bucket[g]] + rank[g] : ~0u;
  }
  __device__ __forceinline__ uint32_t turns() const { return (total + 15u) / 16u; }
  // A bit for each turn with one of the lanes' chosen scenarios (bit g: that of rank[g]).  All lanes.
  __device__ __forceinline__ uint32_t turns_of(uint32_t chosen) const {
    uint32_t turns = 0u;
#pragma unroll
    for (uint32_t g = 0; g < kWindowGroups; ++g)
      if (((chosen >> g) & 1u) != 0u && rank[g] != ~0u) turns |= 1u << (rank[g] >> 4);
    for (int off = 32; off > 0; off >>= 1) turns |= (uint32_t)__shfl_xor((int)turns, off);
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)turns);
  }
  // which: the scenario of the window that the lane's quad takes; false: none.  All lanes.
  __device__ __forceinline__ bool take(uint32_t turn, void* lds, uint32_t& which) const {
    uint16_t* const chosen = (uint16_t*)lds + 64u * kWindowGroups;
    const uint32_t lane = threadIdx.x & 63u;
    __syncthreads();
#pragma unroll
    for (uint32_t g = 0; g < kWindowGroups; ++g)
      if (rank[g] >> 4 == turn) chosen[rank[g] & 15u] = (uint16_t)(kBlock * g + lane);
    __syncthreads();
    const bool exists = 16u * turn + (lane >> 2) < total;
    which = exists ? chosen[lane >> 2] : 0u;
    __syncthreads();
    return exists;
  }
};

// The turn that a workgroup of 16 quads takes, where there is one for each: in ragged batches.
// Turns are a window's longest (0) to its shortest ones.  The windows' longest and shortest
// start first and the ones in between last; every power of two of workgroups in a row has as
// many of the one as of the other (the Thue-Morse sequence), so that a SIMD, which gets
// workgroups some power of two apart, has not only long ones, whatever the batch's size is.
// (With a turn further on from window to window, which gave SIMDs turns of one length: 60,000
// scenarios of powers of two and both policies, 64 chunks, 311 us, now 219, of 128 chunks 591 ->
// 412; the longest first all over: 216, 417, but 60,000 4-D of 250 chunks 1,119 for 995.)
struct WindowTurn {
  uint64_t window;
  uint32_t turn, turns;   // (turns: of the window)
};
__host__ __device__ constexpr WindowTurn window_turn(uint64_t n, uint32_t block) {
  const uint32_t whole = (uint32_t)(n / kWindow);   // (blocks are 32-bit numbers)
  if (block >= (uint64_t)whole * kWindowTurns)   // the last window, not a whole one
    return {whole, block % kWindowTurns, (uint32_t)(n % kWindow + 15u) / 16u};
  const uint32_t slot = block / whole;
  uint32_t odd = slot ^ slot >> 4;
  odd = odd ^ odd >> 2;
  odd = (odd ^ odd >> 1) & 1u;
  return {block % whole, odd != 0u ? kWindowTurns - 1u - (slot >> 1) : slot >> 1, kWindowTurns};
}

// What a window's order is made from.
struct WindowScenario {
  uint32_t D, length;   // (length: events)
  bool in_range;   // (dimensions and chunks; what else makes a scenario invalid is not looked at)
};
__device__ __forceinline__ WindowScenario window_scenario(const themis_batch_t& b, uint64_t i) {
  WindowScenario w;
  w.D = b.ndims[i];
  const uint32_t C = b.chunks[i];
  const bool one_phase = b.collective_type && b.collective_type[i] != THEMIS_COLL_ALL_REDUCE;
  w.in_range = w.D - 1u < (uint32_t)kMaxDims && C - 1u < b.max_chunks;
  w.length = w.in_range ? C * w.D * (one_phase ? 1u : 2u) : 1u;
  return w;
}
// Is a batch to be taken in turns of its windows, not 16 neighbours at a time?  Where 64 of its
// scenarios do not all have the same length (the same answer in every workgroup), and where
// finding the order, some 10 us beside other work, is little beside a turn (60,000 scenarios,
// neighbours / turns, us: powers of two of up to 8 chunks 46 / 50, 16 77 / 69 and on four
// dimensions 78 / 82, 24 109 / 91 and 110 / 110, 32 135 / 116 and 140 / 131; any NPU counts on three
// dimensions 8 35 / 50, 24 74 / 85, 32 93 / 100).
__device__ __forceinline__ bool in_turns(const themis_batch_t& b) {
  const uint32_t length = window_scenario(b, (b.n - 1u) * (threadIdx.x & 63u) / 63u).length;
  const bool differ = __builtin_amdgcn_ballot_w64(length != (uint32_t)__builtin_amdgcn_readfirstlane((int)length)) != 0ull;
  return b.max_chunks > 24u && differ;
}
// Does it have an NPU count that is not a power of two?
__device__ __forceinline__ bool other_counts(const themis_batch_t& b, uint64_t i, uint32_t D) {
  uint32_t more = 0u;   // bits beside the lowest one of each
#pragma unroll
  for (uint32_t k = 0; k < (uint32_t)kMaxDims; ++k) {
    const uint32_t p = b.npus[(size_t)k * b.n + i];
    more |= k < D ? p & (p - 1u) : 0u;
  }
  return more != 0u;
}

// Are three quarters of a batch of other counts, by 64 of its scenarios?  (The same answer in
// every workgroup.)
__device__ __forceinline__ bool mostly_others(const themis_batch_t& b) {
  const uint64_t i = (b.n - 1u) * (threadIdx.x & 63u) / 63u;
  return __builtin_popcountll(__builtin_amdgcn_ballot_w64(other_counts(b, i, b.ndims[i]))) >= 48;
}

// What is left marked of a window's scenarios of four dimensions, or of the others (four), in
// turns.  The kernels before leave those of other counts, or powers of two beside such.  What is
// left as a rule comes first where that is a part of the scenarios, so a few of them share
// turns.  The longest first.  From the inputs alone, as every workgroup of the window has to
// find the same turns whatever the others have done already.  All lanes.
enum class LeftFirst { kAll, kOthers, kPow2 };
struct MarkedWindow {
  uint32_t length[kWindowGroups];   // as in QuadWindow
  __device__ __forceinline__ MarkedWindow(const themis_batch_t& b, uint64_t from, bool four) {
#pragma unroll
    for (uint32_t g = 0; g < kWindowGroups; ++g) {
      const uint64_t j = from + kBlock * g + (threadIdx.x & 63u);
      const WindowScenario w = window_scenario(b, j < b.n ? j : b.n - 1u);
      length[g] = j < b.n && w.in_range && (w.D == 4u) == four ? w.length : 0u;
    }
  }
  // marked: bit g of the lane's scenarios.  Are there any among them?
  __device__ __forceinline__ bool any(uint32_t marked) const {
    uint32_t here = 0u;
#pragma unroll
    for (uint32_t g = 0; g < kWindowGroups; ++g) here |= length[g] != 0u ? 1u << g : 0u;
    return __builtin_amdgcn_ballot_w64((here & marked) != 0u) != 0ull;
  }
  // turns: those with marks
  __device__ __forceinline__ QuadWindow order(const themis_batch_t& b, uint64_t from, LeftFirst first, uint32_t marked,
                                              void* lds, uint32_t& turns) {
    const uint32_t most = 2u * (uint32_t)kMaxDims * b.max_chunks;
    if (first != LeftFirst::kAll) {
#pragma unroll
      for (uint32_t g = 0; g < kWindowGroups; ++g) {
        const uint64_t j = from + kBlock * g + (threadIdx.x & 63u), at = j < b.n ? j : b.n - 1u;
        const bool sooner = other_counts(b, at, b.ndims[at]) == (first == LeftFirst::kOthers);
        // (one less: the longest of the rest are not in the bucket of the shortest that come first)
        length[g] = length[g] == 0u ? 0u : sooner ? length[g] + most : max(length[g] - 1u, 1u);
      }
    }
    const QuadWindow w(first != LeftFirst::kAll ? 2u * most : most, lds, length);
    turns = w.turns_of(marked);
    return w;
  }
};

}  // namespace themis
