// Many orders of one scenario (the searches): a wavefront whose 64 lanes
// evaluate the same scenario under different per-chunk orders shares one table
// of everything that depends on a chunk's order alone, so the ring loop of
// themis_ring.hpp runs on it whatever the NPU counts are, and lower bounds of
// the completion time come from a few additions.
//
// LDS of a wavefront (SharedTable), entry (rank of the order) * 8 + (stages
// behind the chunk):
//   step      what the stage does, as in ring_loop's table
//   time      its duration
// and per order rank
//   load[k]   time the chunk keeps dimension k busy
//   head[k]   time of its stages before the first one on k
//   tail[k]   time of its stages after the last one on k
//   serial    time of all its stages
#pragma once

#include "themis_wave.hpp"

namespace themis {

struct SharedTable {
  double time[kWaveOrders * 8u];
  uint16_t step[kWaveOrders * 8u];
  float4 load[kWaveOrders], head[kWaveOrders], tail[kWaveOrders];
  float serial[kWaveOrders];
  uint8_t rank_of[32];   // order rank of the permutation with lexicographic index j
};

struct SharedSetup {
  double t_min;      // smallest stage time
  double t_max;      // no schedule of C chunks takes longer than C * t_max
  bool ok;           // the ring loop can run on the table
  bool turns;        // it has entries that stand for two stages (see ring_loop)
  // where a chunk waits first: bits 0 and 1 of the dimension, a bit per order
  // rank, and the class there, four bits per dimension (all chunks start with
  // the same size)
  uint32_t first_dim[2], first_class;
};

// The model ring_loop<kShared> runs on.  at(c): rank of chunk c's order, asked
// once for every chunk in ascending order.
template <typename RankAt>
struct SharedModel {
  const SharedTable& tab;
  const SharedSetup& setup;
  int ctype;
  RankAt& at;
  __device__ __forceinline__ SharedModel(const SharedTable& t, const SharedSetup& u, int type, RankAt& a)
      : tab(t), setup(u), ctype(type), at(a) {}
  __device__ __forceinline__ uint32_t epack() const { return 0u; }
  __device__ __forceinline__ uint64_t ranks() const { return 0ull; }
  __device__ __forceinline__ bool rs_only() const { return ctype == THEMIS_COLL_REDUCE_SCATTER; }
  __device__ __forceinline__ bool one_phase() const { return ctype != THEMIS_COLL_ALL_REDUCE; }
  __device__ __forceinline__ uint32_t rank_at(uint32_t c) const { return at(c) & 31u; }
  __device__ __forceinline__ uint32_t first_dim(uint32_t rank) const {
    return ((setup.first_dim[0] >> rank) & 1u) | ((setup.first_dim[1] >> rank) & 1u) << 1;
  }
  __device__ __forceinline__ uint32_t first_class(uint32_t k) const { return (setup.first_class >> (4u * k)) & 15u; }
  __device__ __forceinline__ double stage_time(uint32_t at) const { return tab.time[at]; }
  __device__ __forceinline__ double t_min(uint32_t) const { return setup.t_min; }
};

// Fills the table for all orders of the scenario (all 64 lanes are here and
// have the same arguments; a barrier of the caller's follows).  kTurns: with entries that
// stand for two stages where the queues are Smallest-Chunk-First.
template <bool kTurns>
__device__ __forceinline__ SharedSetup shared_table(const Scenario& s, double chunk, bool scf,
                                                    SharedTable& tab) {
  const uint32_t D = (uint32_t)s.D, lane = lane_id();
  const bool gather = s.ctype == THEMIS_COLL_ALL_GATHER;
  const bool both = s.ctype == THEMIS_COLL_ALL_REDUCE;
  // the orders of D dimensions, read as orders of four
  uint32_t code = ring_order_of_rank(lane % kWaveOrders);
  const uint64_t orders = __builtin_amdgcn_ballot_w64(
      lane < kWaveOrders && (code >> (2u * D)) == (0xe4u >> (2u * D)));
  WaveTables t;
  wave_tables(s, chunk, scf, (uint32_t)orders, t, false);
  const uint32_t phase = lane >= kWaveOrders ? 1u : 0u, rank = lane - (phase ? kWaveOrders : 0u);
  const bool mine = lane < 2u * kWaveOrders && ((orders >> rank) & 1ull) != 0ull;
  double total = 0.0;
  if (mine) {
    float before = 0.0f, sum = 0.0f;
    if (phase == (gather ? 1u : 0u))
      tab.load[rank] = tab.head[rank] = tab.tail[rank] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
    for (int k = 0; k < kMaxDims; ++k)
      if (k < (int)D) { sum += (float)t.time[k]; total = total + t.time[k]; }
    if (both) total = total + total;
    for (uint32_t p = 0; p < D; ++p) {
      const int k = (int)((code >> (2u * p)) & 3u);
      const double time = sel4(k, t.time[0], t.time[1], t.time[2], t.time[3]);
      const uint32_t next = sel4(k, t.next[0], t.next[1], t.next[2], t.next[3]);
      const uint32_t stage = both ? (phase ? 2u * D - 1u - p : p) : (gather ? D - 1u - p : p);
      if (both || phase == (gather ? 1u : 0u)) {
        tab.time[rank * 8u + stage] = time;
        const uint32_t step = ((next >> kWaveDimShift) << 4) | ((next >> kWaveClassShift) & 15u) |
                              ((next & kWaveFinished) ? kRingFinished : 0u) | (phase << 9);
        // (the last Reduce-Scatter stands for the first All-Gather too, with what that one does)
        const bool turns = kTurns && both && scf;
        if (!(turns && phase == 0u && p + 1u == D)) tab.step[rank * 8u + stage] = (uint16_t)(step | 1u << 10);
        if (turns && phase != 0u && p + 1u == D) tab.step[rank * 8u + stage - 1u] = (uint16_t)(step | 2u << 10);
      }
      if (phase == (gather ? 1u : 0u)) {
        const float tk = (float)time;
        ((float*)&tab.load[rank])[k] = both ? 2.0f * tk : tk;
        // (a stand-alone All-Gather runs from the order's last field to its first)
        const float after = fmaxf(sum - before - tk, 0.0f);
        ((float*)&tab.head[rank])[k] = gather ? after : before;
        ((float*)&tab.tail[rank])[k] = both || gather ? before : after;
        before += tk;
      }
    }
    if (phase == (gather ? 1u : 0u)) tab.serial[rank] = both ? 2.0f * sum : sum;
  }
  if (lane < factorial_u32(D)) {
    const uint32_t given = nth_permutation_code(D, lane);
    tab.rank_of[lane] = (uint8_t)ring_order_rank(gather ? reverse_code(given, (int)D) : given, D);
  }
  for (int off = 32; off > 0; off >>= 1) {
    const double other = __shfl_xor(total, off);
    total = other > total ? other : total;
  }
  SharedSetup r;
  const bool starts = mine && phase == (gather ? 1u : 0u);
  const uint32_t kf = (code >> (gather ? 2u * D - 2u : 0u)) & 3u, shift = gather ? kWaveOrders : 0u;
  r.first_class = 0u;
#pragma unroll
  for (uint32_t k = 0; k < (uint32_t)kMaxDims; ++k) {
    const uint64_t on = __builtin_amdgcn_ballot_w64(starts && kf == k);
    if (on != 0ull)
      r.first_class |= ((uint32_t)__builtin_amdgcn_readlane((int)t.first_class[k], __builtin_ctzll(on)) & 15u)
                       << (4u * k);
  }
  r.first_dim[0] = (uint32_t)(__builtin_amdgcn_ballot_w64(starts && (kf & 1u) != 0u) >> shift);
  r.first_dim[1] = (uint32_t)(__builtin_amdgcn_ballot_w64(starts && (kf & 2u) != 0u) >> shift);
  r.t_min = t.t_min;
  r.t_max = total;
  r.ok = t.normal && t.few_classes;
  r.turns = kTurns && both && scf;
  return r;
}

// The event loop on the table: completion time only.  kTurns: as the table's.  (A second loop in
// the exhaustive search's kernel costs first-in-first-out, which has no turns, 472 -> 480 us.)
template <bool kTurns, typename RankAt>
__device__ __forceinline__ FastResult shared_ring(const Scenario& s, const SharedModel<RankAt>& model, const LaneLds& lds) {
  FastOut none;
  none.queue_order = nullptr;
  none.slots = 0u;
  const uint8_t* const table = (const uint8_t*)model.tab.step;
  if constexpr (kTurns)
    if (first_lane(model.setup.turns ? 1u : 0u) != 0u)
      return ring_loop<true, kNoQueueOrder, false, false, true, true>(s, model, lds, none, table);
  return ring_loop<true, kNoQueueOrder, false, false, true, false>(s, model, lds, none, table);
}

// Lower bound of the completion time of chunks with the given orders: a
// dimension is busy for all of its stages, after the shortest way to it and
// before the shortest way from it; and no chunk is faster than its own stages.
// In single precision, taken down by more than its rounding.
struct SharedBound {
  float4 load = {0.0f, 0.0f, 0.0f, 0.0f};
  float4 head = {3.0e38f, 3.0e38f, 3.0e38f, 3.0e38f}, tail = head;
  float serial = 0.0f;
  // both: an All-Reduce, whose way from a dimension is as long as the way to it
  __device__ __forceinline__ void add(const SharedTable& tab, uint32_t rank, bool both) {
    const float4 l = tab.load[rank], h = tab.head[rank];
    load.x += l.x; load.y += l.y; load.z += l.z; load.w += l.w;
    head.x = fminf(head.x, h.x); head.y = fminf(head.y, h.y);
    head.z = fminf(head.z, h.z); head.w = fminf(head.w, h.w);
    if (!both) {
      const float4 t = tab.tail[rank];
      tail.x = fminf(tail.x, t.x); tail.y = fminf(tail.y, t.y);
      tail.z = fminf(tail.z, t.z); tail.w = fminf(tail.w, t.w);
    }
    serial = fmaxf(serial, tab.serial[rank]);
  }
  // the chunks that the lane `off` away has added
  __device__ __forceinline__ void join(int off, bool both) {
    load.x += __shfl_xor(load.x, off); load.y += __shfl_xor(load.y, off);
    load.z += __shfl_xor(load.z, off); load.w += __shfl_xor(load.w, off);
    head.x = fminf(head.x, __shfl_xor(head.x, off)); head.y = fminf(head.y, __shfl_xor(head.y, off));
    head.z = fminf(head.z, __shfl_xor(head.z, off)); head.w = fminf(head.w, __shfl_xor(head.w, off));
    if (!both) {
      tail.x = fminf(tail.x, __shfl_xor(tail.x, off)); tail.y = fminf(tail.y, __shfl_xor(tail.y, off));
      tail.z = fminf(tail.z, __shfl_xor(tail.z, off)); tail.w = fminf(tail.w, __shfl_xor(tail.w, off));
    }
    serial = fmaxf(serial, __shfl_xor(serial, off));
  }
  __device__ __forceinline__ float value(bool both) const {
    const float4 t = both ? head : tail;
    // (an unused dimension: all zeros)
    const float most = fmaxf(fmaxf(load.x + (head.x + t.x), load.y + (head.y + t.y)),
                             fmaxf(load.z + (head.z + t.z), load.w + (head.w + t.w)));
    return fmaxf(serial, most) * (1.0f - 2.0e-5f);
  }
};

// a / F for F = 1, 2, 6, 24 = 2^shift * (1 or 3), in three instructions for 32-bit a.
struct DivideByOrders {
  uint32_t shift;
  bool three;
  __device__ __forceinline__ explicit DivideByOrders(uint32_t D)
      : shift(D >= 4u ? 3u : D >= 2u ? 1u : 0u), three(D >= 3u) {}
  __device__ __forceinline__ uint32_t operator()(uint32_t a) const {
    const uint32_t x = a >> shift;
    return three ? __umulhi(x, 0xaaaaaaabu) >> 1 : x;
  }
  __device__ __forceinline__ uint64_t operator()(uint64_t a) const {
    const uint64_t x = a >> shift;
    return three ? x / 3u : x;
  }
};

}  // namespace themis
