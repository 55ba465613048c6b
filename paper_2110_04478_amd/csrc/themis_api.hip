// C ABI of the library (see include/themis.h) and the kernels behind it.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdlib>
#include <cstring>
#include <tuple>
#include <utility>

#include "themis.h"
#include "themis_device.hpp"
#include "themis_fast.hpp"
#include "themis_generic.hpp"
#include "themis_ring.hpp"
#include "themis_quad.hpp"
#include "themis_shared.hpp"
#include "themis_table.hpp"
#include "themis_trace.hpp"
#include "themis_trace_quad.hpp"
#include "themis_trace_wave.hpp"
#include "themis_wave.hpp"
#include "themis_window.hpp"

// Scratch of themis_simulate_batch_noalloc: device memory the library itself
// brings along, one copy per GPU that loads the code object.  Host code never
// uses this name as an address; it asks the runtime for the array's device
// address once per device (scratch_of_current_device()).
static __device__ __align__(256) unsigned char scratch[THEMIS_STATIC_SCRATCH_BYTES];

namespace themis {

struct TraceView {
  bool on;
  uint32_t mc;     // collectives per scenario row (1 without a trace)
  uint32_t slots;  // chunk slots per scenario = max_chunks * mc
};

__host__ __device__ inline TraceView trace_view(const themis_batch_t& b) {
  TraceView t;
  t.on = b.n_coll != nullptr;
  t.mc = t.on ? b.max_coll : 1u;
  t.slots = b.max_chunks * t.mc;
  return t;
}

__device__ __forceinline__ double collective_size(const themis_batch_t& b, const TraceView& tv,
                                                  uint64_t i, uint32_t q) {
  return tv.on ? b.coll_size[(size_t)q * b.n + i] : b.size_bytes[i];
}

__device__ __forceinline__ double collective_release(const themis_batch_t& b, const TraceView& tv,
                                                     uint64_t i, uint32_t q) {
  return (tv.on && b.release_time) ? b.release_time[(size_t)q * b.n + i] : 0.0;
}

// Checks the collectives of scenario i (count, sizes, release times).
__device__ __forceinline__ bool collectives_ok(const themis_batch_t& b, const TraceView& tv,
                                               uint64_t i, uint32_t& Q) {
  Q = tv.on ? b.n_coll[i] : 1u;
  if (Q < 1u || Q > tv.mc) { Q = 0; return false; }
  bool ok = true;
  for (uint32_t q = 0; q < Q; ++q) {
    if (!finite_positive(collective_size(b, tv, i, q))) ok = false;
    double r = collective_release(b, tv, i, q);
    if (!(r >= 0.0 && r < inf64())) ok = false;
  }
  return ok;
}

__device__ __forceinline__ bool threshold_ok(double thr, bool rel) {
  return thr >= 0.0 && (!rel || thr < inf64());
}

// A completion time of this bit pattern (a NaN no computation produces) marks
// an evaluation that the LDS kernel leaves to the generic kernel launched
// right behind it.  Keeping the generic path out of the LDS kernels keeps its
// registers and scratch memory out of their budgets.
constexpr uint64_t kLeftToGeneric = 0x7ff8a5a55a5a0001ull;
__device__ __forceinline__ double left_to_generic() { return __longlong_as_double((long long)kLeftToGeneric); }
__device__ __forceinline__ bool is_left_to_generic(double t) {
  return (uint64_t)__double_as_longlong(t) == kLeftToGeneric;
}

// Every call that may hand evaluations over carries a number of its own (host
// counter, never 0); a kernel that marks one raises this word to its call's
// number, and the follow-up kernels of a call return at once while the word is
// below theirs -- then nothing of that call can be marked.  A larger number
// left by another call only costs the scan for marks.
__device__ unsigned long long g_marked_call = 0ull;
__device__ __forceinline__ void mark_left_to_generic(double* slot, unsigned long long call) {
  *slot = left_to_generic();
  atomicMax(&g_marked_call, call);
}
__device__ __forceinline__ bool nothing_marked(unsigned long long call) {
  return *(volatile unsigned long long*)&g_marked_call < call;
}

// HIP takes fewer than 2^32 threads along one direction of a grid.  Kernels with four
// lanes per scenario or evaluation reach that four times as early as those with one
// (64 million scenarios of a sweep under 17 pairs of threshold and scheduler), so their
// workgroups are laid out in rows (Launcher::in_rows); those beyond the last one that is
// wanted find nothing to do.
constexpr uint32_t kGridRow = 1u << 25;
__device__ __forceinline__ uint32_t block_index() { return blockIdx.y * kGridRow + blockIdx.x; }

// Work of some lanes of a wavefront, taken by its quads 16 at a time, the longest
// first: a turn takes as long as its longest.
struct QuadTurns {
  uint64_t left;
  uint32_t place;   // of the lane's own work (all-ones: none)
  __device__ __forceinline__ QuadTurns(uint64_t lanes, uint32_t length) : left(lanes), place(0u) {
    const uint32_t lane = threadIdx.x & 63u;
    for (uint64_t m = lanes; m != 0ull; m &= m - 1ull) {
      const uint32_t j = (uint32_t)__builtin_ctzll(m);
      const uint32_t other = (uint32_t)__builtin_amdgcn_readlane((int)length, (int)j);
      place += other > length || (other == length && j < lane) ? 1u : 0u;
    }
    if (((lanes >> lane) & 1ull) == 0ull) place = ~0u;
  }
  // which: the lane whose work the quad takes; false: none is left for it.  All lanes.
  __device__ __forceinline__ bool take(uint32_t& which) {
    const uint32_t lane = threadIdx.x & 63u;
    const bool chosen = place < kBlock / 4u;
    const uint32_t sent = (uint32_t)__builtin_amdgcn_ds_permute(chosen ? (int)(16u * place) : 4, (int)lane);
    which = (uint32_t)__shfl((int)sent, (int)(lane & ~3u));
    const bool exists = (uint32_t)__builtin_popcountll(left) > lane >> 2;
    left &= ~__builtin_amdgcn_ballot_w64(chosen);
    place = place == ~0u || chosen ? ~0u : place - kBlock / 4u;
    return exists;
  }
};

// ---------------------------------------------------------------------------
// themis_plan_batch: Alg. 1 per scenario (hot-path steps a1-a5).
// ---------------------------------------------------------------------------
// kPerCollective: one lane per (scenario, collective) instead of one per
// scenario -- the tracker starts afresh for every collective (Alg. 1 line 2),
// so the collectives of a trace are planned independently, and a batch of a
// few thousand traces has too few scenarios to fill the GPU.
// One or four wavefronts for 64 of them: the first plans those whose NPU counts are
// powers of two, a lane each, and all of them the others, four lanes each, 16 at a
// time (see plan_waves).  They are workgroups of their own, the first ones of all
// groups before the second ones: as one workgroup of four, whose LDS is held until the
// last of them is through, 65,536 scenarios of 32 chunks took 66 us on other NPU counts
// and 29 on powers of two, now 59 and 26.
constexpr uint32_t kPlanWaves = 4u;
template <bool kPerCollective>
__global__ void __launch_bounds__(kBlock)
plan_kernel(themis_batch_t b, uint8_t* __restrict__ orders, double* __restrict__ loads) {
  // the planner's order table, one entry per lane of the workgroup's first wavefront
  static_assert(kBlock == kPlanOrders, "one table entry per lane");
  __shared__ __attribute__((aligned(16))) uint32_t plan_orders[kPlanOrders * kPlanOrderWords];
  const uint32_t lane = threadIdx.x;
  uint32_t wave = 0u, waves = 1u, group = blockIdx.x;
  if (!kPerCollective) {
    const uint32_t groups = (uint32_t)((b.n + kBlock - 1u) / kBlock);
    if (gridDim.x > groups) waves = kPlanWaves;
    for (; group >= groups; group -= groups) ++wave;
  }
  if (wave == 0u) {   // (the only one that reads it; a wavefront's LDS accesses keep their order)
    plan_order_entry(lane, plan_orders + kPlanOrderWords * lane);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  const TraceView tv = trace_view(b);
  const uint64_t first = (uint64_t)group * kBlock, e = first + lane;
  auto scenario_of = [&](uint64_t at) { return kPerCollective ? at / tv.mc : at; };
  const bool rel = b.threshold_mode == THEMIS_THR_REL;
  // a collective's codes, and from there to the end of its row
  auto pad = [&](uint8_t* r, uint32_t filled) {
    for (uint32_t c = filled; c < b.max_chunks; ++c) r[c] = 0xFFu;
  };
  // rows are written four codes at a time when they are 4-byte aligned
  const bool words = (b.max_chunks & 3u) == 0u;
  auto pad_word = [&](uint8_t* r, uint32_t C, uint32_t acc) -> uint32_t {
    if (words && (C & 3u)) {  // pad the last partial word with unused-slot marks
      acc |= 0xFFFFFFFFu << (8u * (C & 3u));
      ((uint32_t*)r)[C >> 2] = acc;
      return (C | 3u) + 1u;
    }
    return C;
  };
  if (waves > 1u) {   // the others leave at once where all counts are powers of two
    bool other = false;
    if (scenario_of(e) < b.n) {
      const uint32_t D = b.ndims[scenario_of(e)];
#pragma unroll
      for (uint32_t k = 0; k < (uint32_t)kMaxDims; ++k)
        other = other || (k < D && !is_pow2(b.npus[(size_t)k * b.n + scenario_of(e)]));
    }
    if (__builtin_amdgcn_ballot_w64(other) == 0ull) waves = 1u;
    if (wave >= waves) return;
  }
  bool left = false;   // NPU counts that are not powers of two: for the quads below
  uint32_t chunks = 0u;
  if (scenario_of(e) < b.n) {
    const uint64_t i = scenario_of(e);
    const uint32_t q = kPerCollective ? (uint32_t)(e - i * tv.mc) : 0u;
    const Scenario s = load_scenario(b, i);
    const double thr = b.threshold[i];
    uint32_t Q;
    const bool ok = collectives_ok(b, tv, i, Q) && s.valid && threshold_ok(thr, rel);
    uint8_t* r = orders + (size_t)i * tv.slots + (size_t)q * b.max_chunks;
    double load[kMaxDims] = {0.0, 0.0, 0.0, 0.0};
    uint32_t filled = 0u;
    if (ok && q < Q) {
      const double chunk = collective_size(b, tv, i, q) / (double)s.C;
      FastScenario fs;
      left = !fast_eligible(s, chunk, THEMIS_MAX_CHUNKS, fs);
      chunks = s.C;
      if (!left && wave == 0u) {
        uint32_t acc = 0;
        plan_fast(s, fs, b.inter_policy[i] != THEMIS_INTER_BASELINE, rel, thr, load, [&](uint32_t c, uint32_t code) {
          if (words) {
            acc |= code << (8u * (c & 3u));
            if ((c & 3u) == 3u) { ((uint32_t*)r)[c >> 2] = acc; acc = 0; }
          } else {
            r[c] = (uint8_t)code;
          }
        }, plan_orders);
        filled = pad_word(r, s.C, acc);
      }
    }
    if (!left && wave == 0u) {
      pad(r, filled);
      // the tracker of the scenario's last collective (an invalid scenario: NaN)
      if (loads && (!kPerCollective || q == (ok ? Q - 1u : 0u))) {
#pragma unroll
        for (int k = 0; k < kMaxDims; ++k)
          loads[(size_t)k * b.n + i] = ok ? ((k < s.D) ? load[k] : 0.0) : nan64();
      }
    }
  }
  const uint64_t others = __builtin_amdgcn_ballot_w64(left);
  QuadTurns turns(others, chunks);
  for (uint32_t turn = 0; turns.left != 0ull; ++turn) {
    uint32_t which;
    const bool exists = turns.take(which);
    if (turn % waves != wave) continue;
    const uint64_t at = exists ? first + which : first, i = scenario_of(at);
    const uint32_t q = kPerCollective ? (uint32_t)(at - i * tv.mc) : 0u, k = threadIdx.x & 3u;
    const Scenario s = load_scenario(b, i);
    const double chunk = collective_size(b, tv, i, q) / (double)s.C;
    uint8_t* r = orders + (size_t)i * tv.slots + (size_t)q * b.max_chunks;
    double least = chunk, load;
#pragma unroll
    for (int d = 0; d < kMaxDims; ++d)
      if (d < s.D) least = least / (double)s.P[d];
    uint32_t acc = 0u;
    auto emit = [&](uint32_t c, uint32_t code) {
      acc |= code << (8u * (c & 3u));
      if (k != 0u) return;
      if (!words) r[c] = (uint8_t)code;
      else if ((c & 3u) == 3u) { ((uint32_t*)r)[c >> 2] = acc; acc = 0u; }
    };
    const bool themis_on = b.inter_policy[i] != THEMIS_INTER_BASELINE;
    const uint32_t C = exists ? s.C : 0u;
    if (__builtin_amdgcn_ballot_w64(exists && !(least >= 2.2250738585072014e-308)) == 0ull)
      plan_quad<false>(s, chunk, themis_on, rel, b.threshold[i], C, load, emit);
    else
      plan_quad<true>(s, chunk, themis_on, rel, b.threshold[i], C, load, emit);
    if (exists) {
      if (k == 0u) pad(r, pad_word(r, C, acc));
      const uint32_t Q = tv.on ? b.n_coll[i] : 1u;
      if (loads && (!kPerCollective || q + 1u == Q)) loads[(size_t)k * b.n + i] = k < (uint32_t)s.D ? load : 0.0;
    }
  }
}

// One wavefront per scenario and collective: for batches that cannot fill the
// GPU with one lane each (see plan_on_wavefronts).
__global__ void __launch_bounds__(kBlock)
plan_wave_kernel(themis_batch_t b, uint8_t* __restrict__ orders, double* __restrict__ loads) {
  const TraceView tv = trace_view(b);
  const uint64_t i = blockIdx.x / tv.mc;
  const uint32_t q = (uint32_t)(blockIdx.x - i * tv.mc);
  const uint32_t lane = lane_id();
  const Scenario s = load_scenario(b, i);
  const bool rel = b.threshold_mode == THEMIS_THR_REL;
  const double thr = b.threshold[i];
  uint32_t Q;
  const bool ok = collectives_ok(b, tv, i, Q) && s.valid && threshold_ok(thr, rel);
  uint8_t* row = orders + (size_t)i * tv.slots + (size_t)q * b.max_chunks;
  double load[kMaxDims] = {0.0, 0.0, 0.0, 0.0};
  uint32_t filled = 0u;
  if (ok && q < Q) {
    const double chunk = collective_size(b, tv, i, q) / (double)s.C;
    wave_plan(s, chunk, b.inter_policy[i] != THEMIS_INTER_BASELINE, rel, thr, load,
              [&](uint32_t first, uint32_t code) {
                if (first + lane < s.C) row[first + lane] = (uint8_t)code;
              });
    filled = s.C;
  }
  for (uint32_t c = filled + lane; c < b.max_chunks; c += kBlock) row[c] = 0xFFu;
  // the tracker of the scenario's last collective (an invalid scenario: NaN)
  if (loads && q == (ok ? Q - 1u : 0u) && lane < (uint32_t)kMaxDims) {
    const double v = sel4((int)lane, load[0], load[1], load[2], load[3]);
    loads[(size_t)lane * b.n + i] = ok ? ((int)lane < s.D ? v : 0.0) : nan64();
  }
}

// ---------------------------------------------------------------------------
// themis_simulate_batch (hot-path steps a6-a9): LDS fast path, with the
// generic workspace path for the scenarios it does not cover.
// ---------------------------------------------------------------------------
// i: scenario; col: its column of the workspace arrays.
template <bool kEager>
__device__ __forceinline__ void simulate_generic_scenario(const themis_batch_t& b, const TraceView& tv,
                                                          const Scenario& s, uint32_t Q, uint64_t i,
                                                          uint64_t col, const uint8_t* row, bool scf,
                                                          const Workspace& w, const SimOut& out) {
  bool ok = true;
  bool has_release = false;
  // a6: every chunk waits at the dimension of its first stage
  for (uint32_t q = 0; q < Q; ++q) {
    double chunk = collective_size(b, tv, i, q) / (double)s.C;
    double rel = collective_release(b, tv, i, q);
    has_release |= rel > 0.0;
    for (uint32_t c = 0; c < s.C; ++c) {
      uint32_t code = row[(size_t)q * b.max_chunks + c];
      if (!order_code_ok(code, s.D)) ok = false;
      size_t at = (size_t)(q * s.C + c) * w.stride + col;
      w.meta[at] = code << 8;
      w.size[at] = chunk;
      w.arrival[at] = rel;
    }
  }
  if (!ok) { write_invalid(out); return; }
  simulate_generic<kEager>(
      s, Q, scf, w, col,
      [&](uint32_t q) { return collective_size(b, tv, i, q) / (double)s.C; },
      [&](uint32_t q) { return collective_release(b, tv, i, q); }, has_release, out);
}

// This lane's view of its wavefront's LDS block.
template <typename L>
__device__ __forceinline__ LaneLds lane_lds(uint32_t* lds_block) {
  LaneLds lds;
  if constexpr (IsRing<L>::value) {
    lds.base = (uint8_t*)lds_block + L::lane_term_rec(threadIdx.x);
    lds.aux = (uint8_t*)lds_block + L::lane_term_tail(threadIdx.x);
  } else {
    lds.base = (uint8_t*)lds_block + 4u * threadIdx.x;
    lds.aux = nullptr;
  }
  return lds;
}

// The power-of-two event loop that goes with the layout.
template <typename L, int kQueueOrder, bool kBusy, bool kFix>
__device__ __forceinline__ FastResult simulate_pow2(const Scenario& s, const Pow2Model& model,
                                                    const LaneLds& lds, const FastOut& out) {
  if constexpr (IsRing<L>::value) {
    // entries leave one by one: collected dwords become single bytes
    constexpr int kMode = kQueueOrder == kWords ? (int)kBytes : kQueueOrder;
    return simulate_ring<kMode, kBusy, kFix>(s, model, lds, out);
  } else {
    return simulate_fast<L, kQueueOrder, kBusy, kFix, Pow2Model>(s, model, lds, out);
  }
}

// All-ones from entry `used` of a row of `row_len` entries on.
__device__ __forceinline__ void pad_row(uint8_t* row, uint32_t used, uint32_t row_len, int entry_bytes) {
  uint32_t at = used * (uint32_t)entry_bytes;
  const uint32_t end = row_len * (uint32_t)entry_bytes;
  for (; at < end && ((uintptr_t)(row + at) & 7u) != 0u; ++at) row[at] = 0xFFu;
  for (; at + 8u <= end; at += 8u) *(uint64_t*)(row + at) = ~0ull;
  for (; at < end; ++at) row[at] = 0xFFu;
}

// The order codes of a scenario, four chunks at a time: each lane of the quad looks at one
// of them.  take(code): what is to be known about it, 18 bits; visit(c, taken): by every
// lane, in the order of the chunks.  C: 0 where there is no scenario.
// (Each lane looking at all four: 61 vector and 53 scalar instructions a chunk, a third of that here,
// and the event loop of a 3-D chunk is some 300; with the planner 65,536 3-D scenarios of 64 chunks
// 234 -> 219 us, 20,001 4-D ones of 250 chunks 890 -> 818.)
template <typename Take, typename Visit>
__device__ __forceinline__ void quad_codes(const themis_batch_t& b, const uint8_t* orders, uint64_t i, uint32_t C,
                                           Take take, Visit visit) {
  const uint32_t k = threadIdx.x & 3u;
  const uint8_t* const row = orders + (size_t)i * b.max_chunks;
  uint32_t code = k < C ? row[k] : 0u;
  for (uint32_t c = 0; c < C; c += 4u) {
    const uint32_t now = code;
    if (c + 4u + k < C) code = row[c + 4u + k];   // (on its way meanwhile)
    const uint32_t mine = c + k < C ? take(now) : ~0u;
    const uint32_t of[4] = {quad_lane<0>(mine), quad_lane<1>(mine), quad_lane<2>(mine), quad_lane<3>(mine)};
#pragma unroll
    for (uint32_t j = 0; j < 4u; ++j)
      if (of[j] != ~0u) visit(c + j, of[j]);
  }
}
// Is it a permutation of dimensions 0 .. D - 1?
__device__ __forceinline__ bool quad_code_ok(uint32_t code, uint32_t D) {
  const uint32_t c8 = code | (0xe4u & ~((1u << (2u * D)) - 1u));   // (the others behind them)
  return (code >> (2u * D)) == 0u &&
         ((1u << (c8 & 3u)) | (1u << ((c8 >> 2) & 3u)) | (1u << ((c8 >> 4) & 3u)) | (1u << (c8 >> 6))) == 15u;
}

// What a quad writes about its scenario (mark: left to the kernels that follow,
// which write everything).
template <int kQueueOrder>
__device__ __forceinline__ void quad_outputs(const themis_batch_t& b, uint64_t i, bool done, bool mark,
                                             const QuadResult& r, double* t_done, uint8_t* row, int entry_bytes,
                                             double* busy, unsigned long long call) {
  const uint32_t k = threadIdx.x & 3u;
  if (mark) {
    if (k == 0u) mark_left_to_generic(t_done + i, call);
    return;
  }
  if (k == 0u) t_done[i] = done ? r.t_done : nan64();
  if (busy) busy[(size_t)k * b.n + i] = done ? r.busy : nan64();
  if (kQueueOrder != kNoQueueOrder) pad_row(row, done ? r.started : 0u, 2u * b.max_chunks, entry_bytes);
}

// One scenario (i) per quad, of up to kDims dimensions and L::kCap chunks, whatever its NPU
// counts are (QuadTable).  What the event loop does not take is marked, unless it is
// marked already (marked); malformed codes are for the caller's kernel or the generic
// one, and so are invalid scenarios unless the caller leaves them here (invalid_too).
// Returns whether it is (still) marked.  All lanes of the wavefront; lds: QuadTable::kBytes.
template <typename L, uint32_t kDims, int kQueueOrder>
__device__ __forceinline__ bool quad_table_turn(const themis_batch_t& b, const uint8_t* __restrict__ orders,
                                                double* __restrict__ t_done, void* __restrict__ queue_order,
                                                int entry_bytes, double* __restrict__ busy, uint64_t i, bool exists,
                                                bool marked, bool invalid_too, void* lds, unsigned long long call) {
  using Table = QuadTable<L, kDims>;
  const uint32_t k = threadIdx.x & 3u;
  const Scenario s = load_scenario(b, i);
  const double S = b.size_bytes[i];
  const bool ok = s.valid && finite_positive(S), invalid = exists && !ok && invalid_too;
  exists = exists && ok;
  const uint32_t D = (uint32_t)s.D;
  const bool gather = s.ctype == THEMIS_COLL_ALL_GATHER;
  uint32_t bad = 0u, used = 0u;
  auto order_of = [&](uint32_t code) {
    return quad_order(gather ? reverse_code(code, s.D) : code, D) % Table::kOrders;
  };
  if (exists)
    for (uint32_t c16 = k; c16 < s.C; c16 += 16u) {
      uint32_t code[4];
#pragma unroll
      for (uint32_t j = 0; j < 4u; ++j) code[j] = orders[(size_t)i * b.max_chunks + min(c16 + 4u * j, s.C - 1u)];
#pragma unroll
      for (uint32_t j = 0; j < 4u; ++j) {
        if (!quad_code_ok(code[j], D)) bad = 1u;
        used |= 1u << order_of(code[j]);
      }
    }
  const bool runs = exists && quad_sum(bad) == 0u;
  used = runs ? quad_or(used) : 0u;
  const Table model(s, S / (double)s.C, b.intra_policy[i] == THEMIS_INTRA_SCF, used, lds);
  QuadQueue<L> queue(lds);
  quad_codes(b, orders, i, runs ? s.C : 0u,
             [&](uint32_t code) { return Table::state_of(order_of(code), gather ? 1u : 0u) << 9 | (code & 3u) << 16; },
             [&](uint32_t c, uint32_t taken) {
               if (taken >> 16 == k) queue.add(c | (taken & 0xffffu));
             });
  uint8_t* const row = queue_order ? (uint8_t*)queue_order + ((size_t)i * kMaxDims + k) * 2u * b.max_chunks * (uint32_t)entry_bytes
                                   : nullptr;
  const uint32_t stages = s.ctype == THEMIS_COLL_ALL_REDUCE ? 2u * D : D;
  const QuadResult r = simulate_quad<L, kQueueOrder != kNoQueueOrder>(
      model, queue, model.cls0, runs ? stages * s.C : 0u, model.t_min, [&](uint32_t e, uint32_t entry) {
        if (kQueueOrder == kShorts) ((uint16_t*)row)[e] = (uint16_t)entry;
        else row[e] = (uint8_t)entry;
      });
  const bool done = runs && r.ok;
  if (invalid || (exists && (done || !marked)))
    quad_outputs<kQueueOrder>(b, i, done, !done && !invalid, r, t_done, row, entry_bytes, busy, call);
  __syncthreads();
  return exists && !done;
}

// As L, with registers for two wavefronts on a SIMD and no more: for batches that are all
// resident so, whose time is that of the fullest SIMD.  With room for three the GPU gives
// some SIMDs three and others one, or not, after what ran before: behind plan_kernel with
// its four wavefronts 100,003 4-D scenarios of 64 chunks took 486 us, 128,299 of 61 chunks
// 448; so they take 405 and 355, as behind a planner of one wavefront.
template <typename L>
struct TwoPerSimd : L {
  static constexpr uint32_t kWavesPerSimd = 2;
};

// Do the scenarios of a wavefront of lanes that are powers of two go with the others?
__device__ __forceinline__ bool lanes_few(bool in_range, bool others) {
  return __builtin_amdgcn_ballot_w64(others) != 0ull &&
         __builtin_popcountll(__builtin_amdgcn_ballot_w64(in_range && !others)) <= 16;
}

template <typename L, int kQueueOrder, bool kBusy, bool kFix>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(L::kWavesPerSimd)))
simulate_kernel(themis_batch_t b, const uint8_t* __restrict__ orders,
                double* __restrict__ t_done, void* __restrict__ queue_order, int entry_bytes,
                double* __restrict__ busy, unsigned long long hand_over) {
  __shared__ __attribute__((aligned(8))) uint32_t lds_block[L::kLaneWords * kBlock];
  // (a third of a SIMD's 512 registers per lane, and a few, see TwoPerSimd)
  if constexpr (L::kWavesPerSimd == 2u) asm volatile("" : : : "v175");
  // (a lane beyond the batch stays for the exchanges between lanes)
  const uint64_t at = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  const bool exists = at < b.n;
  const uint64_t i = exists ? at : b.n - 1u;
  const Scenario s = load_scenario(b, i);
  const bool scf = b.intra_policy[i] == THEMIS_INTRA_SCF;
  const double S = b.size_bytes[i];
  const bool ok = s.valid && finite_positive(S);
  FastScenario fs;
  const bool eligible = fast_eligible(s, S / (double)s.C, L::kCap, fs) && ok && exists;
  // NPU counts that are not powers of two: four lanes each at the end, up to three
  // dimensions, else left to the follow-up kernel; with them the other scenarios
  // of the wavefront where those are few (one round of 16 is cheaper than the lanes' loop)
  // (in_range, others: as the other wavefronts of the window see the scenario)
  const bool in_range = exists && b.ndims[i] - 1u < (uint32_t)kMaxDims && s.C - 1u < b.max_chunks;
  const bool others = in_range && other_counts(b, i, b.ndims[i]);
  const bool few = lanes_few(in_range, others);
  const bool fast = eligible && !few;
  const bool tables = in_range && b.ndims[i] < 4u && (others || few);

  // Queue orders of a wavefront whose 64 scenarios all exist are staged
  // transposed inside the wavefront's own block of the output (kStagedBytes)
  // and put in place once the wavefront is through: a lane appends an entry to
  // one of its four rows at every event, and with the rows in place the
  // partly written lines of all resident wavefronts do not fit the L2, so they
  // go to memory several times over.
  // dwords per row that the last step holds in registers (a row has up to
  // kCap / 2).  Up to 64 chunks: with the four wavefronts per CU of the
  // 128-chunk layout the rows written in place do better (3.14 against 3.44 ms
  // for 262,144 scenarios of 126 chunks).
  constexpr uint32_t kStagedWords = L::kCap / 2u < 32u ? L::kCap / 2u : 32u;
  const uint32_t rows_bytes = (uint32_t)kMaxDims * 2u * b.max_chunks * (uint32_t)entry_bytes;
  const bool staged = kQueueOrder == kWords && queue_order != nullptr &&
                      (b.max_chunks >> 1) <= kStagedWords &&
                      (uint64_t)(blockIdx.x + 1u) * kBlock <= b.n;  // the same for all lanes
  enum { kRowsStaged = 1, kRowsAllOnes = 2, kRowsNotMine = 3 };
  uint32_t rows = kRowsNotMine;
  uint32_t executed[kMaxDims] = {0u, 0u, 0u, 0u};

  SimOut out;
  out.t_done = t_done + i;
  out.busy = busy ? busy + i : nullptr;
  out.busy_stride = b.n;
  out.entry_bytes = entry_bytes;
  out.slots = b.max_chunks;
  out.queue_order = (kQueueOrder != kNoQueueOrder && queue_order)
      ? (void*)((uint8_t*)queue_order + (size_t)i * rows_bytes) : nullptr;
  // an invalid scenario: NaN / all-ones (its rows at the end, if rows are staged in the block)
  auto invalid = [&]() {
    SimOut o = out;
    if (staged) o.queue_order = nullptr;
    write_invalid(o);
    rows = kRowsAllOnes;
  };

  bool left = false;
  if (exists) do {
    if (!ok) { invalid(); break; }
    const uint8_t* row = orders + (size_t)i * b.max_chunks;
    if (fast) {
      const LaneLds lds = lane_lds<L>(lds_block);
      // order codes -> chunk words (mask 0, Reduce-Scatter phase)
      bool codes_ok = true;
      if ((b.max_chunks & 3u) == 0u) {
        const uint32_t* row4 = (const uint32_t*)row;
        for (uint32_t c4 = 0; c4 < s.C; c4 += 4u) {
          uint32_t v = row4[c4 >> 2];
#pragma unroll
          for (uint32_t j = 0; j < 4u; ++j) {
            if (c4 + j < s.C) {
              uint32_t code = (v >> (8u * j)) & 0xffu;
              codes_ok = codes_ok && order_code_ok(code, s.D);
              L::init_chunk(lds, c4 + j, stored_code(s, fs, code), fs.state0);
            }
          }
        }
      } else {
        for (uint32_t c = 0; c < s.C; ++c) {
          uint32_t code = row[c];
          codes_ok = codes_ok && order_code_ok(code, s.D);
          L::init_chunk(lds, c, stored_code(s, fs, code), fs.state0);
        }
      }
      if (!codes_ok) { invalid(); break; }
      FastOut fo;
      fo.queue_order = (uint8_t*)out.queue_order;
      fo.slots = b.max_chunks;
      // staged: the same address for all lanes plus a 32-bit offset
      FastOut so;
      so.queue_order = (uint8_t*)queue_order + (size_t)blockIdx.x * kBlock * rows_bytes;
      so.slots = b.max_chunks;
      so.lane_offset = IsRing<L>::value ? threadIdx.x : 4u * threadIdx.x;
      so.staging_bytes = (uint32_t)kBlock * rows_bytes;
      FastResult r;
      if constexpr (kQueueOrder == kWords) {
        r = staged ? simulate_pow2<L, kStagedBytes, kBusy, kFix>(s, Pow2Model(s, fs, scf), lds, so)
                   : simulate_pow2<L, kWords, kBusy, kFix>(s, Pow2Model(s, fs, scf), lds, fo);
      } else {
        r = simulate_pow2<L, kQueueOrder, kBusy, kFix>(s, Pow2Model(s, fs, scf), lds, fo);
      }
      if (r.ok) {
        t_done[i] = r.t_done;
        if (busy) {
#pragma unroll
          for (int k = 0; k < kMaxDims; ++k) busy[(size_t)k * b.n + i] = r.busy[k];
        }
        if (staged) {
          rows = kRowsStaged;
#pragma unroll
          for (int k = 0; k < kMaxDims; ++k) executed[k] = r.executed[k];
        } else if (kQueueOrder != kNoQueueOrder && out.queue_order) {
          for (int k = 0; k < kMaxDims; ++k)
            for (uint32_t e = r.executed[k]; e < 2u * b.max_chunks; ++e)
              fo.queue_order[(uint32_t)k * 2u * b.max_chunks + e] = 0xFFu;
        }
        break;
      }
    }
    left = true;
  } while (false);

  if constexpr (kQueueOrder == kWords) {
    if (staged) {
      // every lane fetches its own rows from the staging order (64 lanes read
      // 256 contiguous bytes per dword), waits until the whole wavefront has
      // all of them in registers, and writes them where they belong, with
      // all-ones from the first unused entry on
      const uint32_t wpr = b.max_chunks >> 1;  // dwords per row
      // the entries a lane fetches were stored by other lanes of its wavefront
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
      const uint32_t* from =
          (const uint32_t*)((uint8_t*)queue_order + (size_t)blockIdx.x * kBlock * rows_bytes) + threadIdx.x;
      uint32_t q[kMaxDims][kStagedWords];
      if constexpr (IsRing<L>::value) {
        // the ring loop stages single bytes, entry j of a row at byte 64 * j +
        // lane: the four lanes of a quad fetch the dwords of entries 4w .. 4w+3
        // (one each, the quad's four bytes of that entry) and exchange them, a
        // 4 x 4 byte transpose inside the quad
        const uint32_t sub = threadIdx.x & 3u;
        const uint32_t* from4 = (const uint32_t*)((uint8_t*)queue_order +
                                                  (size_t)blockIdx.x * kBlock * rows_bytes) +
                                sub * 16u + (threadIdx.x >> 2);
        // byte `sub` of the first operand's dword into byte 0, of the second's into byte 1
        const uint32_t pick = sub * 0x0101u + 0x0400u;
#pragma unroll
        for (uint32_t k = 0; k < (uint32_t)kMaxDims; ++k)
#pragma unroll
          for (uint32_t w = 0; w < kStagedWords; ++w)
            q[k][w] = w < wpr ? from4[(size_t)(k * wpr + w) * kBlock] : 0xffffffffu;
        // (the wait states a lane-crossing read asks for after a change of exec)
        asm volatile("s_waitcnt vmcnt(0)\n\ts_nop 4" ::: "memory");
#pragma unroll
        for (uint32_t k = 0; k < (uint32_t)kMaxDims; ++k)
#pragma unroll
          for (uint32_t w = 0; w < kStagedWords; ++w) {
            // lane a of the quad holds entry 4w + a: everybody takes byte `sub`
            // of all four.  One block per dword, three temporaries: left to the
            // compiler, the 128 dwords and its temporaries no longer fit the
            // registers of three wavefronts per SIMD.
            uint32_t t0, t1, t2;
            asm volatile(
                "v_mov_b32_dpp %[t0], %[q] quad_perm:[0,0,0,0] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
                "v_mov_b32_dpp %[t1], %[q] quad_perm:[1,1,1,1] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
                "v_mov_b32_dpp %[t2], %[q] quad_perm:[2,2,2,2] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
                "v_perm_b32 %[t0], %[t1], %[t0], %[pick]\n\t"
                "v_mov_b32_dpp %[t1], %[q] quad_perm:[3,3,3,3] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
                "v_perm_b32 %[t1], %[t1], %[t2], %[pick]\n\t"
                "v_perm_b32 %[q], %[t1], %[t0], %[join]"
                : [q] "+v"(q[k][w]), [t0] "=&v"(t0), [t1] "=&v"(t1), [t2] "=&v"(t2)
                : [pick] "v"(pick), [join] "s"(0x05040100u));
            if (rows != kRowsStaged) q[k][w] = 0xffffffffu;
          }
      } else {
#pragma unroll
        for (uint32_t k = 0; k < (uint32_t)kMaxDims; ++k)
#pragma unroll
          for (uint32_t w = 0; w < kStagedWords; ++w)
            q[k][w] = (w < wpr && rows == kRowsStaged) ? from[(size_t)(k * wpr + w) * kBlock] : 0xffffffffu;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      }
      if (rows != kRowsNotMine) {
        uint32_t* to = (uint32_t*)((uint8_t*)queue_order + (size_t)i * rows_bytes);
        // four dwords per store where the rows allow it: a quarter of the
        // memory transactions of this step
        const bool quads = (wpr & 3u) == 0u && ((uintptr_t)queue_order & 15u) == 0u;
        // rows without an unused entry (every dimension ran all 2 * slots
        // operations: an All-Reduce of `slots` chunks on four dimensions) need no marks
        bool full_rows = rows == kRowsStaged;
#pragma unroll
        for (uint32_t k = 0; k < (uint32_t)kMaxDims; ++k) full_rows = full_rows && executed[k] == 2u * b.max_chunks;
        const bool marks = __builtin_amdgcn_ballot_w64(!full_rows) != 0ull;  // the same for all lanes
#pragma unroll
        for (uint32_t k = 0; k < (uint32_t)kMaxDims; ++k)
#pragma unroll
          for (uint32_t w4 = 0; w4 < kStagedWords; w4 += 4u) {
            uint32_t v[4];
#pragma unroll
            for (uint32_t j = 0; j < 4u; ++j) {
              const uint32_t w = w4 + j;
              v[j] = w < kStagedWords ? q[k][w] : 0xffffffffu;
              if (marks) {
                // entries of this dword that are in use, 0..4; all-ones above them
                const int left = min(max((int)executed[k] - (int)(4u * w), 0), 4);
                v[j] |= (uint32_t)(0xffffffffull << (8 * left));
              }
            }
            if (quads) {
              if (w4 < wpr) *(uint4*)(to + k * wpr + w4) = make_uint4(v[0], v[1], v[2], v[3]);
            } else {
#pragma unroll
              for (uint32_t j = 0; j < 4u; ++j)
                if (w4 + j < wpr) to[k * wpr + w4 + j] = v[j];
            }
          }
      }
    }
  }
  // (what ran in the lanes' loop and stalled there goes on to the generic path)
  if (left && !tables) mark_left_to_generic(t_done + i, hand_over);
  using L3 = LayoutQuad<L::kCap, 12u, 3u>;
  static_assert(QuadTable<L3, 3>::kBytes <= sizeof(lds_block), "the tables fit the lanes' block");
  const uint64_t own = __builtin_amdgcn_ballot_w64(tables);
  if (own != 0ull) {
    // The wavefronts of a window that have nothing else share the turns of all of them.  (One
    // whose lanes ran has staged queue orders in the rows of all its scenarios, so nobody
    // else may write any of those; it takes its own.)
    const uint64_t window = blockIdx.x / kWindowGroups, from = window * kWindow, first = (uint64_t)blockIdx.x * kBlock;
    uint32_t sharing = 0u;
    uint32_t lengths[kWindowGroups];
#pragma unroll
    for (uint32_t g = 0; g < kWindowGroups; ++g) {
      const uint64_t j = from + kBlock * g + threadIdx.x;
      const bool there = j < b.n;
      const WindowScenario w = window_scenario(b, there ? j : b.n - 1u);
      const bool other = other_counts(b, there ? j : b.n - 1u, w.D), range = there && w.in_range;
      lengths[g] = w.length;
      const bool few_here = lanes_few(range, range && other), member = range && few_here && w.D < 4u;
      if (__builtin_amdgcn_ballot_w64(member) != 0ull) sharing |= 1u << g;
      if (!member) lengths[g] = 0u;
    }
    const QuadWindow shared(2u * (uint32_t)kMaxDims * b.max_chunks, lds_block, lengths);
    const uint32_t of = max((uint32_t)__builtin_popcount(sharing), 1u);
    const uint32_t me = (uint32_t)__builtin_popcount(sharing & ((1u << blockIdx.x % kWindowGroups) - 1u));
    // (workgroups go to the XCDs in turn: not every window's longest to the same one)
    uint32_t turn = (me + (uint32_t)window) % of;
    QuadTurns alone(few ? 0ull : own, tables ? window_scenario(b, i).length : 0u);
    while (few ? turn < shared.turns() : alone.left != 0ull) {
      uint32_t which;
      const bool there = few ? shared.take(turn, lds_block, which) : alone.take(which);
      turn += of;
      quad_table_turn<L3, 3, kQueueOrder>(b, orders, t_done, queue_order, entry_bytes, busy,
                                          there ? (few ? from : first) + which : first, there, false, false, lds_block,
                                          hand_over);
    }
  }
}

// Four lanes per scenario (themis_quad.hpp).  kOthers: scenarios of up to three
// dimensions whose NPU counts are not powers of two are taken here as well, by tables of
// their own; else, and on four dimensions, they are left marked.
// A wavefront takes 16 neighbours, with others among them those of up to three dimensions by
// tables, whatever their counts; in ragged batches (in_turns()) one turn of a window: of the
// others, or of the rest.
template <typename L, int kQueueOrder, bool kFix, bool kOthers>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(L::kWavesPerSimd)))
simulate_quad_kernel(themis_batch_t b, const uint8_t* __restrict__ orders, double* __restrict__ t_done,
                     void* __restrict__ queue_order, int entry_bytes, double* __restrict__ busy,
                     unsigned long long hand_over) {
  using L3 = LayoutQuad<L::kCap, 12u, 3u>;
  constexpr uint32_t kLdsBytes = kOthers && QuadTable<L3, 3>::kBytes > QuadPow2<L, kFix>::kBytes ? QuadTable<L3, 3>::kBytes : QuadPow2<L, kFix>::kBytes;
  __shared__ uint64_t lds_block[(kLdsBytes + 7u) / 8u];
  const uint32_t k = threadIdx.x & 3u, block = block_index();
  if ((uint64_t)block * L::kQuads >= b.n) return;   // (in the grid's last row)
  const bool ragged = in_turns(b);
  // a quad without a scenario stays: the wavefront leaves the event loop as a whole
  uint64_t i = (uint64_t)block * L::kQuads + (threadIdx.x >> 2);
  bool exists = i < b.n, runs_rest = true;
  const WindowTurn mine = ragged ? window_turn(b.n, block) : WindowTurn{};
  const uint64_t from = mine.window * kWindow;
  const uint32_t turn = mine.turn, blocks = mine.turns;
  uint32_t turns_of_rest = 0u;
  // of the others or of the rest (0: not one of them)
  auto lengths_of = [&](bool others, uint32_t (&lengths)[kWindowGroups]) {
#pragma unroll
    for (uint32_t g = 0; g < kWindowGroups; ++g) {
      const uint64_t j = from + kBlock * g + threadIdx.x, at = j < b.n ? j : b.n - 1u;
      const WindowScenario w = window_scenario(b, at);
      const bool other = kOthers && w.in_range && w.D < 4u && other_counts(b, at, w.D);
      lengths[g] = j < b.n && other == others ? w.length : 0u;
    }
  };
  if (ragged) {
    uint32_t lengths[kWindowGroups];
    lengths_of(false, lengths);
    const QuadWindow rest(2u * (uint32_t)kMaxDims * b.max_chunks, lds_block, lengths);
    turns_of_rest = rest.turns();
    uint32_t which;
    exists = rest.take(turn, lds_block, which);
    i = from + which;
    runs_rest = turn < turns_of_rest;
  }
  if (!exists) i = b.n - 1u;
  bool tables = false;
  if (runs_rest) {
    const Scenario s = load_scenario(b, i);
    const uint32_t D = (uint32_t)s.D;
    const double S = b.size_bytes[i];
    FastScenario fs;
    const bool ok = s.valid && finite_positive(S) && exists;
    const bool eligible = fast_eligible(s, S / (double)s.C, L::kCap, fs) && ok;
    const bool others = kOthers && !ragged && __builtin_amdgcn_ballot_w64(ok && !eligible && D < 4u) != 0ull;
    tables = others && ok && D < 4u;
    // a few powers of two beside other counts that are left go with those (alone in a wavefront
    // they take as long as a full one: 2,100 3-D scenarios of 65 chunks and any NPU counts,
    // eleven of them powers of two, 262 -> 143 us, 20,000 of 100 chunks 626 -> 441)
    const bool few = __builtin_popcountll(__builtin_amdgcn_ballot_w64(eligible && !tables)) <= 16 &&
                     __builtin_amdgcn_ballot_w64(ok && !eligible && (D == 4u || !kOthers)) != 0ull;
    const bool fast = eligible && !tables && !few;
    if (!others || __builtin_amdgcn_ballot_w64(exists && !tables) != 0ull) {
      QuadQueue<L> queue(lds_block);
      uint32_t bad = 0u;
      // (a lane takes the chunks that start on its own dimension)
      quad_codes(b, orders, i, fast ? s.C : 0u,
                 [&](uint32_t code) {
                   if (!quad_code_ok(code, D)) bad = 1u;
                   return ((quad_row(D) + quad_order(stored_code(s, fs, code), D)) & 31u) << 9 |
                          (fs.gather ? 1u << L::kPhaseBit : 0u) | (code & 3u) << 16;
                 },
                 [&](uint32_t c, uint32_t taken) {
                   if (taken >> 16 == k) queue.add(c | (taken & 0xffffu));
                 });
      const bool runs = fast && quad_sum(bad) == 0u;
      if (!runs) queue.any = false;
      const Pow2Model pow2(s, fs, b.intra_policy[i] == THEMIS_INTRA_SCF);
      uint8_t* const row = queue_order ? (uint8_t*)queue_order + ((size_t)i * kMaxDims + k) * 2u * b.max_chunks * (uint32_t)entry_bytes
                                       : nullptr;
      QuadResult r{nan64(), nan64(), 0u, false};
      if (__builtin_amdgcn_ballot_w64(runs) != 0ull) r = simulate_quad<L, kQueueOrder != kNoQueueOrder>(
          QuadPow2<L, kFix>(s, pow2, k, lds_block), queue, (uint32_t)(pow2.ranktab >> (4u * (fs.state0 & 15u))) & 15u,
          runs ? (pow2.one_phase() ? D : 2u * D) * s.C : 0u, pow2.t_min(D),
          [&](uint32_t e, uint32_t entry) {
            if (kQueueOrder == kShorts) ((uint16_t*)row)[e] = (uint16_t)entry;
            else row[e] = (uint8_t)entry;
          });
      const bool malformed = fast && !runs, done = runs && r.ok;
      if (exists && !tables)
        quad_outputs<kQueueOrder>(b, i, done, ok && !malformed && !done, r, t_done, row, entry_bytes, busy, hand_over);
    }
  }
  if constexpr (kOthers) {
    if (ragged) {
      // (the longest of them last, see window_turn(); the two kinds have a turn more than there
      // are workgroups, or not)
      const bool one_more = turn == 0u && runs_rest;
      if (!runs_rest || one_more) {
        uint32_t lengths[kWindowGroups];
        lengths_of(true, lengths);
        const QuadWindow turns(2u * (uint32_t)kMaxDims * b.max_chunks, lds_block, lengths);
        uint32_t which;
        const bool there = turns.take(runs_rest ? blocks - turns_of_rest : blocks - 1u - turn, lds_block, which);
        if (__builtin_amdgcn_ballot_w64(there) != 0ull)
          quad_table_turn<L3, 3, kQueueOrder>(b, orders, t_done, queue_order, entry_bytes, busy, from + which, there, false,
                                              true, lds_block, hand_over);
      }
    } else if (__builtin_amdgcn_ballot_w64(tables) != 0ull) {
      __syncthreads();
      quad_table_turn<L3, 3, kQueueOrder>(b, orders, t_done, queue_order, entry_bytes, busy, i, tables, false, false,
                                          lds_block, hand_over);
    }
  }
}

// One wavefront per scenario (themis_wave.hpp): single collectives of up to 64 *
// kWords chunks in batches too small to fill the GPU with one lane per scenario.
// kExact: what the event loop does not take (a stage too short to move the
// clock, sizes outside the normal range) is evaluated right here, and nothing
// follows this kernel: for the smallest batches, where a second launch costs
// more than the registers.  Else it is left marked to the follow-up kernel.
template <uint32_t kWords, bool kQueue, bool kExact>
__global__ void __launch_bounds__(kBlock)
simulate_wave_kernel(themis_batch_t b, const uint8_t* __restrict__ orders, double* __restrict__ t_done,
                     void* __restrict__ queue_order, int entry_bytes, double* __restrict__ busy,
                     unsigned long long hand_over) {
  using Lds = WaveLds<kWords>;
  using ExactLds = WaveExactLds<kExact ? kWords : 1u>;
  __shared__ union Block {
    Lds events;
    ExactLds exact;
    __device__ Block() {}
  } block;
  Lds& lds = block.events;
  const uint64_t i = blockIdx.x;
  const uint32_t lane = lane_id();
  const Scenario s = load_scenario(b, i);
  const bool scf = b.intra_policy[i] == THEMIS_INTRA_SCF;
  const double S = b.size_bytes[i];
  const uint32_t C = s.C;
  const uint32_t row_len = 2u * b.max_chunks;
  uint8_t* rows = queue_order ? (uint8_t*)queue_order + (size_t)i * kMaxDims * row_len * (uint32_t)entry_bytes
                              : nullptr;
  auto put = [&](uint32_t k, uint32_t at, uint32_t entry) {
    if (kQueue) {
      const uint32_t e = k * row_len + at;
      if (entry_bytes == 1) rows[e] = (uint8_t)entry;
      else ((uint16_t*)rows)[e] = (uint16_t)entry;
    }
  };
  WaveResult r;
#pragma unroll
  for (int k = 0; k < kMaxDims; ++k) { r.busy[k] = nan64(); r.executed[k] = 0u; }
  r.t_done = nan64();
  bool ok = s.valid && finite_positive(S);
  if (ok) {
    const uint8_t* row = orders + (size_t)i * b.max_chunks;
    const double chunk = S / (double)C;
    const WaveOutcome outcome =
        wave_simulate<kWords, kQueue>(s, chunk, scf, lds, [&](uint32_t c) { return (uint32_t)row[c]; }, r);
    ok = outcome != WaveOutcome::kMalformed;
    if (ok) {
      const bool done = outcome == WaveOutcome::kDone;
      if (kQueue && done) {
#pragma unroll
        for (uint32_t k = 0; k < (uint32_t)kMaxDims; ++k)
          for (uint32_t e = lane; e < r.executed[k]; e += kBlock) {
            const uint32_t rec = lds.log[k][e];
            put(k, e, ((rec & kWaveIdMask) << 1) | ((rec >> kWaveStateShift) >= kWaveOrders ? 1u : 0u));
          }
      }
      if (!done) {
        if constexpr (kExact) {
          __syncthreads();
          r = wave_exact<kWords>(s, chunk, scf, block.exact, [&](uint32_t c) { return (uint32_t)row[c]; },
                                 [&](uint32_t k, uint32_t at, uint32_t entry) {
                                   if (lane == 0u) put(k, at, entry);
                                 });
          ok = r.ok;
        } else {
          if (lane == 0u) mark_left_to_generic(t_done + i, hand_over);
          return;
        }
      }
    }
  }
  if (lane == 0u) t_done[i] = ok ? r.t_done : nan64();
  if (busy && lane < (uint32_t)kMaxDims)
    busy[(size_t)lane * b.n + i] = ok ? sel4((int)lane, r.busy[0], r.busy[1], r.busy[2], r.busy[3]) : nan64();
  if (kQueue) {
#pragma unroll
    for (uint32_t k = 0; k < (uint32_t)kMaxDims; ++k)
      for (uint32_t e = (ok ? r.executed[k] : 0u) + lane; e < row_len; e += kBlock) put(k, e, 0xFFFFu);
  }
}

// Second kernel of themis_simulate_batch: the scenarios the LDS kernel marked.
// kLdsSlots > 0: the per-chunk arrays (20 bytes per chunk) live in LDS, laid
// out like the workspace with the 64 lanes as columns; for batches of at most
// kLdsSlots chunk slots per scenario, which then need no workspace at all.
// LDS a generic pass needs for kLdsSlots chunk slots per lane, in bytes.
constexpr size_t generic_lds_bytes(uint32_t lds_slots) {
  return lds_slots ? (size_t)((lds_slots * kBlock * 5u + 1u) / 2u) * sizeof(double) : 0u;
}

template <uint32_t kLdsSlots>
__device__ __forceinline__ void simulate_generic_lane(
    const themis_batch_t& b, const uint8_t* __restrict__ orders, double* __restrict__ t_done,
    void* __restrict__ queue_order, int entry_bytes, double* __restrict__ busy, const Workspace& w, uint64_t i) {
  const TraceView tv = trace_view(b);
  const uint64_t col = kLdsSlots ? threadIdx.x : i;
  Scenario s = load_scenario(b, i);
  const bool scf = b.intra_policy[i] == THEMIS_INTRA_SCF;
  uint32_t Q;
  collectives_ok(b, tv, i, Q);  // marked scenarios passed this check already
  SimOut out;
  out.t_done = t_done + i;
  out.busy = busy ? busy + i : nullptr;
  out.busy_stride = b.n;
  out.entry_bytes = entry_bytes;
  out.slots = tv.slots;
  out.queue_order = queue_order
      ? (void*)((uint8_t*)queue_order + (size_t)i * kMaxDims * 2u * tv.slots * entry_bytes)
      : nullptr;
  // beyond the LDS variant's chunk count the arrays need the caller's workspace
  if (!kLdsSlots && !w.meta) { write_invalid(out); return; }
  simulate_generic_scenario<(kLdsSlots > 0)>(b, tv, s, Q, i, col, orders + (size_t)i * tv.slots,
                                             scf, w, out);
}

template <uint32_t kLdsSlots>
__global__ void __launch_bounds__(kBlock)
simulate_generic_kernel(themis_batch_t b, const uint8_t* __restrict__ orders,
                        double* __restrict__ t_done, void* __restrict__ queue_order,
                        int entry_bytes, double* __restrict__ busy, Workspace w,
                        unsigned long long call) {
  __shared__ double lds_block[kLdsSlots ? generic_lds_bytes(kLdsSlots) / sizeof(double) : 1u];
  if (nothing_marked(call)) return;
  if (kLdsSlots) w = carve_workspace(lds_block, kBlock, kLdsSlots);
  // a few workgroups walk all groups of scenarios: most have nothing marked
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < b.n; i += (uint64_t)gridDim.x * kBlock)
    if (is_left_to_generic(t_done[i]))
      simulate_generic_lane<kLdsSlots>(b, orders, t_done, queue_order, entry_bytes, busy, w, i);
}

constexpr size_t max_bytes(size_t a, size_t b) { return a > b ? a : b; }
constexpr uint32_t kNoGeneric = 0xffffffffu;

// Everything that follows the LDS kernel of themis_simulate_batch, in one launch: what
// is marked in quads on tables of its own, then by the generic loop (kGeneric: its
// chunk slots in LDS, 0: arrays in the workspace, kNoGeneric: none).  An item of the
// workgroups' work is a share of a window: every `shares`th of the turns of its scenarios of
// four dimensions, or of the others.  It looks at the window once and leaves where nothing
// is marked.  A scenario belongs to one item, whatever is marked, so what one workgroup finds
// does not depend on the others.  (Up to 64 chunks the kernels before have taken what has other
// counts on up to three dimensions, and leave a few powers of two that were beside those.)
// (Before, every turn of a window was an item that looked at all of it, and turns were of all
// its scenarios; us, then / now: 1,048,576 4-D scenarios of 64 chunks, one of other counts 2,448 /
// 2,306, 10,000 6,054 / 2,640, every eighth 15,032 / 4,494; 65,537, every eighth 1,434 / 662;
// 100,000 3-D of 128 chunks, every eighth 2,474 / 995, all 1,908 / 1,898.)
// (On four dimensions the tables of 24 orders and up to 48 sizes per dimension
// take 37 KiB per wavefront, four wavefronts per CU.)
__host__ __device__ inline uint32_t follow_up_shares_of_others(uint32_t shares, uint32_t cap) {
  return cap > 64u ? shares : (shares + 7u) / 8u;
}
__host__ __device__ inline uint64_t follow_up_items(uint64_t n, uint32_t cap, uint32_t shares) {
  return (n + kWindow - 1u) / kWindow * (shares + follow_up_shares_of_others(shares, cap));
}
template <int kQueueOrder, uint32_t kCap, uint32_t kGeneric>
__global__ void __launch_bounds__(kBlock)
simulate_follow_up_kernel(themis_batch_t b, const uint8_t* __restrict__ orders,
                          double* __restrict__ t_done, void* __restrict__ queue_order,
                          int entry_bytes, double* __restrict__ busy, Workspace w, uint32_t shares,
                          unsigned long long call) {
  using L4 = LayoutQuad<kCap, 48u>;
  using L3 = LayoutQuad<kCap, 12u, 3u>;
  constexpr size_t kBytes_ = max_bytes(QuadTable<L4, 4>::kBytes, kGeneric == kNoGeneric ? 0u : generic_lds_bytes(kGeneric));
  static_assert(QuadTable<L3, 3>::kBytes <= QuadTable<L4, 4>::kBytes, "one block for both");
  __shared__ double lds_block[(kBytes_ + 7u) / 8u];
  if (nothing_marked(call)) return;
  constexpr uint32_t kLdsSlots = kGeneric == kNoGeneric ? 0u : kGeneric;
  if (kLdsSlots) w = carve_workspace(lds_block, kBlock, kLdsSlots);
  const uint32_t lane = threadIdx.x;
  const uint64_t windows = (b.n + kWindow - 1u) / kWindow, items = follow_up_items(b.n, kCap, shares);
  const LeftFirst others_first = mostly_others(b) ? LeftFirst::kAll : LeftFirst::kOthers;
  for (uint64_t item = blockIdx.x; item < items; item += gridDim.x) {
    const uint64_t from = item % windows * kWindow;
    const uint32_t place = (uint32_t)(item / windows);
    const bool four = place < shares;
    const uint32_t share = four ? place : place - shares, step = four ? shares : follow_up_shares_of_others(shares, kCap);
    MarkedWindow window(b, from, four);
    uint32_t marked = 0u;
#pragma unroll
    for (uint32_t g = 0; g < kWindowGroups; ++g) {
      const uint64_t j = from + kBlock * g + lane;
      if (is_left_to_generic(t_done[j < b.n ? j : b.n - 1u])) marked |= 1u << g;
    }
    if (!window.any(marked)) continue;
    uint32_t turns;
    const QuadWindow order = window.order(b, from, !four && kCap <= 64u ? LeftFirst::kPow2 : others_first, marked, lds_block, turns);
    for (; turns != 0u; turns &= turns - 1u) {
      const uint32_t turn = (uint32_t)__builtin_ctz(turns);
      if (turn % step != share) continue;
      uint32_t which;
      const bool there = order.take(turn, lds_block, which);
      const uint64_t i = from + which;   // (from, where there is none)
      const bool exists = there && is_left_to_generic(t_done[i]);
      bool left = four ? quad_table_turn<L4, 4, kQueueOrder>(b, orders, t_done, queue_order, entry_bytes, busy, i, exists,
                                                             true, false, lds_block, call)
                       : quad_table_turn<L3, 3, kQueueOrder>(b, orders, t_done, queue_order, entry_bytes, busy, i, exists,
                                                             true, false, lds_block, call);
      left = left && (lane & 3u) == 0u;
      if (kGeneric != kNoGeneric) {
        __syncthreads();
        if (left) simulate_generic_lane<kLdsSlots>(b, orders, t_done, queue_order, entry_bytes, busy, w, i);
        __syncthreads();
      }
    }
  }
}

// The sweeps' passes over marked evaluations whose NPU counts are not powers of
// two (themis_table.hpp), one lane each: first the variant for at most 8 distinct
// order codes, then (kWide) the one for any number of them; what they cannot take
// stays marked for the generic pass.
// kVariant: 0 tables for at most 8 order codes (64 chunks), 1 any number of
// codes (64 chunks), 2 the same for up to 128 chunks, 3 and 4 16-bit chunk
// records for up to 256 and 512 chunks.
template <int kVariant>
struct TableVariant {
  using L = typename std::conditional<kVariant == 0, LayoutTable,
            typename std::conditional<kVariant == 1, LayoutTableWide,
            typename std::conditional<kVariant == 2, LayoutTableWide128,
            typename std::conditional<kVariant == 3, LayoutTablePacked<256>,
                                      LayoutTablePacked<512>>::type>::type>::type>::type;
};

template <int kVariant>
constexpr size_t table_lds_bytes() {
  if constexpr (kVariant < 0) return 0u;
  else return (size_t)TableVariant<kVariant>::L::kLaneWords * kBlock * sizeof(uint32_t);
}

// ---------------------------------------------------------------------------
// themis_simulate_batch for traces (several collectives sharing the queues):
// the ranked-list path of themis_trace.hpp, else the generic path.
// ---------------------------------------------------------------------------
// kExtras: the batch carries release times or fixed delays (one switch for
// both keeps the number of variants down).  call != 0: only the traces that the
// call's simulate_trace_wave_kernel has left marked.
template <bool kLdsBitmaps, bool kExtras>
__global__ void __launch_bounds__(kBlock)
simulate_trace_kernel(themis_batch_t b, const uint8_t* __restrict__ orders,
                      double* __restrict__ t_done, void* __restrict__ queue_order,
                      int entry_bytes, double* __restrict__ busy, Workspace w, bool have_ws,
                      uint8_t* __restrict__ trace_area, TraceLayout tl, unsigned long long call) {
  __shared__ uint32_t lds_block[(kLdsBitmaps ? kTraceLdsWordsBitmaps : kTraceLdsWords) * kBlock];
  if (call != 0ull && nothing_marked(call)) return;
  uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= b.n || (call != 0ull && !is_left_to_generic(t_done[i]))) return;
  const TraceView tv = trace_view(b);
  Scenario s = load_scenario(b, i);
  const bool scf = b.intra_policy[i] == THEMIS_INTRA_SCF;
  uint32_t Q;
  bool ok = collectives_ok(b, tv, i, Q) && s.valid;

  SimOut out;
  out.t_done = t_done + i;
  out.busy = busy ? busy + i : nullptr;
  out.busy_stride = b.n;
  out.entry_bytes = entry_bytes;
  out.slots = tv.slots;
  out.queue_order = queue_order
      ? (void*)((uint8_t*)queue_order + (size_t)i * kMaxDims * 2u * tv.slots * entry_bytes)
      : nullptr;
  if (!ok) { write_invalid(out); return; }

  const uint8_t* row = orders + (size_t)i * tv.slots;
  bool fast = trace_area != nullptr && tl.bytes != 0u && Q <= tl.Q;
  uint32_t epack = 0;
  FastScenario fs0;
  fs0.state0 = 0u; fs0.rs_only = false; fs0.gather = false;
  if (fast) {
    TraceRegion rg;
    rg.base = trace_area + (size_t)i * tl.bytes;
    rg.t = tl;
    // Every collective in the range where halvings are exact: sizes by
    // exponent arithmetic.  Otherwise (NPU counts that are not powers of two)
    // one division at a time, with size ranks per (dimension, phase, order)
    // under Smallest-Chunk-First as long as they fit the lists.
    bool has_release = false, divide = false;
    for (uint32_t q = 0; q < Q; ++q) {
      const double chunk = collective_size(b, tv, i, q) / (double)s.C;
      divide = divide || !fast_eligible(s, chunk, THEMIS_MAX_CHUNKS, fs0);
    }
    // (division mode ranks every (phase, order) of a dimension: more lists than the masks of halving mode)
    fast = fast && (!divide || !scf ||
                    Q * trace_division_lists((uint32_t)s.D, s.ctype != THEMIS_COLL_ALL_REDUCE) <= tl.R);
    for (uint32_t q = 0; q < Q; ++q) {
      const double chunk = collective_size(b, tv, i, q) / (double)s.C;
      fast_eligible(s, chunk, THEMIS_MAX_CHUNKS, fs0);   // (collective type, initial state; base and epack if exact)
      epack = fs0.epack;
      rg.CH(q) = divide ? chunk : fs0.base;  // resident size at mask 0
      if (kExtras) {
        const double release = collective_release(b, tv, i, q);
        rg.REL(q) = release;
        has_release = has_release || release > 0.0;
      }
    }
    bool codes_ok = true;
    if (fast) {
      for (uint32_t q = 0; q < Q; ++q)
        for (uint32_t c = 0; c < s.C; ++c) {
          const uint32_t code = row[(size_t)q * b.max_chunks + c];
          codes_ok = codes_ok && order_code_ok(code, s.D);
          rg.W(q * s.C + c) = trace_word(stored_code(s, fs0, code), fs0.state0);
        }
      if (!codes_ok) { write_invalid(out); return; }
      LaneLds lds;
      lds.base = (uint8_t*)lds_block + 4u * threadIdx.x;
      double T, z[kMaxDims];
      uint32_t ex[kMaxDims];
      // All-Reduces under one policy on one kind of NPU counts get a loop
      // compiled for exactly that when the whole wavefront is in the case
      const bool all_reduce = __builtin_amdgcn_ballot_w64(fs0.rs_only || fs0.state0 != 0u) == 0ull;
      const uint64_t lanes_scf = __builtin_amdgcn_ballot_w64(scf);
      const uint64_t lanes_divide = __builtin_amdgcn_ballot_w64(divide);
      const uint64_t lanes = __builtin_amdgcn_ballot_w64(true);
      int known = kTraceAnyLane;
      if (all_reduce && (lanes_scf == 0ull || lanes_scf == lanes) &&
          (lanes_divide == 0ull || lanes_divide == lanes))
        known = (lanes_scf ? kTraceKnownScf : 0) | (lanes_divide ? kTraceKnownDivide : 0);
      bool done;
#define THEMIS_TRACE_RUN(KNOWN)                                                                  \
  done = simulate_trace_fast<kLdsBitmaps, kExtras, kExtras, kExtras, KNOWN>(                     \
      s, Q, epack, fs0.state0, fs0.rs_only, scf, divide, has_release, rg, lds, out, T, z, ex)
      switch (known) {
        case 0: THEMIS_TRACE_RUN(0); break;
        case kTraceKnownScf: THEMIS_TRACE_RUN(kTraceKnownScf); break;
        case kTraceKnownDivide: THEMIS_TRACE_RUN(kTraceKnownDivide); break;
        case kTraceKnownScf | kTraceKnownDivide: THEMIS_TRACE_RUN(kTraceKnownScf | kTraceKnownDivide); break;
        default: THEMIS_TRACE_RUN(kTraceAnyLane); break;
      }
#undef THEMIS_TRACE_RUN
      if (done) {
        t_done[i] = T;
        if (busy) {
#pragma unroll
          for (int k = 0; k < kMaxDims; ++k) busy[(size_t)k * b.n + i] = z[k];
        }
        if (out.queue_order) {
          for (int k = 0; k < kMaxDims; ++k)
            for (uint32_t e = ex[k]; e < 2u * tv.slots; ++e) put_entry(out, k, e, 0xFFFFu);
        }
        return;
      }
    }
  }
  if (!have_ws) { write_invalid(out); return; }
  simulate_generic_scenario<false>(b, tv, s, Q, i, i, row, scf, w, out);
}

// Four lanes per trace (themis_trace_quad.hpp): traces released together, NPU counts
// that are powers of two, up to `dims` dimensions; what is left is marked.
// follow_up: only what an earlier launch of the call, for fewer dimensions, has marked.
template <bool kPut>
__global__ void __launch_bounds__(kBlock)
simulate_trace_quad_kernel(themis_batch_t b, const uint8_t* __restrict__ orders, double* __restrict__ t_done,
                           void* __restrict__ queue_order, int entry_bytes, double* __restrict__ busy,
                           uint8_t* __restrict__ trace_area, uint32_t stride, uint32_t dims, bool follow_up,
                           unsigned long long call) {
  extern __shared__ __attribute__((aligned(16))) uint8_t trace_lds[];
  if (follow_up && nothing_marked(call)) return;
  const TraceView tv = trace_view(b);
  const uint32_t k = threadIdx.x & 3u;
  const uint64_t first = (uint64_t)block_index() * (kBlock / 4u), at = first + (threadIdx.x >> 2);
  const bool exists = at < b.n && (!follow_up || is_left_to_generic(t_done[at]));
  if (__builtin_amdgcn_ballot_w64(exists) == 0ull) return;
  const uint64_t i = at < b.n ? at : b.n - 1u;
  const Scenario s = load_scenario(b, i);
  const bool scf = b.intra_policy[i] == THEMIS_INTRA_SCF;
  const uint32_t Q = b.n_coll[i];
  bool ok = s.valid && Q >= 1u && Q <= tv.mc;
  FastScenario fs;
  bool takes = (uint32_t)s.D <= dims, valid = true;
  double smallest = inf64();
  for (uint32_t q = k; ok && q < Q; q += 4u) {
    const double size = collective_size(b, tv, i, q), chunk = size / (double)s.C;
    valid = valid && finite_positive(size);
    takes = takes && fast_eligible(s, chunk, THEMIS_MAX_CHUNKS, fs);
    smallest = min_f64(smallest, chunk);
  }
  fast_eligible(s, ok ? collective_size(b, tv, i, 0u) / (double)s.C : 1.0, THEMIS_MAX_CHUNKS, fs);
  ok = ok && quad_min_u32(valid ? 1u : 0u) != 0u;
  takes = quad_min_u32(takes ? 1u : 0u) != 0u;
  smallest = quad_min_f64(smallest);
  const bool runs = exists && ok && takes;
  const TraceQuadLayout l = trace_quad_layout(tv.slots, dims, tv.mc);
  const uint8_t* const row = orders + (size_t)i * tv.slots;
  const bool dwords = (b.max_chunks & 3u) == 0u && ((uintptr_t)orders & 3u) == 0u;
  uint8_t* const entries = queue_order ? (uint8_t*)queue_order + ((size_t)i * kMaxDims + k) * 2u * tv.slots * (uint32_t)entry_bytes
                                       : nullptr;
  const TraceQuadResult r = simulate_trace_quad<kPut>(
      s, fs, runs ? Q : 0u, scf, smallest, l, trace_lds, trace_area + (size_t)first * stride, stride,
      [&](uint32_t q, uint32_t c) {
        const uint8_t* at_c = row + (size_t)q * b.max_chunks + c;
        if (dwords) return *(const uint32_t*)at_c;
        uint32_t v = 0u;
        for (uint32_t j = 0; j < 4u && c + j < s.C; ++j) v |= (uint32_t)at_c[j] << (8u * j);
        return v;
      },
      [&](uint32_t q) { return collective_size(b, tv, i, q) / (double)s.C; },
      [&](uint32_t e, uint32_t entry) {
        if (entry_bytes == 2) ((uint16_t*)entries)[e] = (uint16_t)entry;
        else entries[e] = (uint8_t)entry;
      });
  if (!exists) return;
  const bool done = runs && r.ok;
  if (ok && !done) {   // (malformed codes: written by the kernel that follows)
    if (k == 0u) mark_left_to_generic(t_done + i, call);
    return;
  }
  if (k == 0u) t_done[i] = done ? r.t_done : nan64();
  if (busy) busy[(size_t)k * b.n + i] = done ? r.busy : nan64();
  if (kPut) pad_row(entries, done ? r.started : 0u, 2u * tv.slots, entry_bytes);
}

// One wavefront per trace (themis_trace_wave.hpp), lds_bytes of LDS: traces that
// need more, or that the event loop does not take (sizes outside the normal
// range, a stage too short to move the clock, a release at the very instant of
// a completion), are left marked.  follow_up: only what an earlier launch of the
// call, with less LDS, has marked.
template <bool kLog>
__global__ void __launch_bounds__(kBlock)
simulate_trace_wave_kernel(themis_batch_t b, const uint8_t* __restrict__ orders, double* __restrict__ t_done,
                           void* __restrict__ queue_order, int entry_bytes, double* __restrict__ busy,
                           uint32_t lds_bytes, bool follow_up, unsigned long long call) {
  extern __shared__ __attribute__((aligned(16))) uint8_t trace_lds[];
  const uint64_t i = blockIdx.x;
  if (follow_up && (nothing_marked(call) || !is_left_to_generic(t_done[i]))) return;
  const TraceView tv = trace_view(b);
  const uint32_t lane = lane_id();
  const Scenario s = load_scenario(b, i);
  const bool scf = b.intra_policy[i] == THEMIS_INTRA_SCF;
  const bool gather = s.ctype == THEMIS_COLL_ALL_GATHER;
  const uint32_t Q = b.n_coll[i];
  bool ok = s.valid && Q >= 1u && Q <= tv.mc;
  bool exact = true, releases = false, sizes_ok = true;
  double smallest = inf64(), largest = 0.0;
  for (uint32_t q = lane; ok && q < Q; q += kBlock) {
    const double size = collective_size(b, tv, i, q), release = collective_release(b, tv, i, q);
    sizes_ok = sizes_ok && finite_positive(size) && release >= 0.0 && release < inf64();
    releases = releases || release > 0.0;
    const double chunk = size / (double)s.C;
    FastScenario fs;
    exact = exact && fast_eligible(s, chunk, THEMIS_MAX_CHUNKS, fs);
    smallest = min_f64(smallest, chunk);
    largest = -min_f64(-largest, -chunk);
  }
  ok = ok && __builtin_amdgcn_ballot_w64(!sizes_ok) == 0ull;
  exact = __builtin_amdgcn_ballot_w64(!exact) == 0ull;
  releases = uniform(releases);
  for (int off = 32; off > 0; off >>= 1) {
    smallest = min_f64(smallest, __shfl_xor(smallest, off));
    largest = -min_f64(-largest, -__shfl_xor(largest, off));
  }
  const uint32_t row_len = 2u * tv.slots;
  uint8_t* const rows = kLog ? (uint8_t*)queue_order + (size_t)i * kMaxDims * row_len * (uint32_t)entry_bytes : nullptr;
  WaveResult r;
#pragma unroll
  for (int k = 0; k < kMaxDims; ++k) { r.busy[k] = nan64(); r.executed[k] = 0u; }
  r.t_done = nan64();
  if (ok) {
    WaveOutcome outcome = WaveOutcome::kNotTaken;
    const TraceWaveLayout l = trace_wave_layout(Q * s.C, (uint32_t)s.D, Q, scf, !exact);
    bool takes = l.bytes <= lds_bytes && lds_offset(trace_lds) == 0u &&
                 trace_wave_lists((uint32_t)s.D, Q, scf, !exact) <= kTraceMaxRanks;
    if (!exact) {
      for (int k = 0; k < s.D; ++k) {
        if (gather) largest = largest * (double)s.P[k];
        else smallest = smallest / (double)s.P[k];
      }
      takes = takes && uniform(smallest >= 2.2250738585072014e-308 && largest < inf64());
    }
    if (takes) {
      const uint8_t* row = orders + (size_t)i * tv.slots;
      auto run = [&](auto divide) {
        return trace_wave_simulate<kLog, decltype(divide)::value>(
            s, Q, scf, releases, smallest, l, trace_lds,
            [&](uint32_t q, uint32_t c) { return (uint32_t)row[(size_t)q * b.max_chunks + c]; },
            [&](uint32_t q) { return collective_size(b, tv, i, q) / (double)s.C; },
            [&](uint32_t q) { return collective_release(b, tv, i, q); }, rows, row_len,
            entry_bytes == 2 ? 1u : 0u, r);
      };
      outcome = exact ? run(std::false_type{}) : run(std::true_type{});
    }
    if (outcome == WaveOutcome::kNotTaken) {
      if (lane == 0u) mark_left_to_generic(t_done + i, call);
      return;
    }
    ok = outcome == WaveOutcome::kDone;
  }
  if (lane == 0u) t_done[i] = ok ? r.t_done : nan64();
  if (busy && lane < (uint32_t)kMaxDims)
    busy[(size_t)lane * b.n + i] = ok ? sel4((int)lane, r.busy[0], r.busy[1], r.busy[2], r.busy[3]) : nan64();
  if (kLog) {
#pragma unroll
    for (uint32_t k = 0; k < (uint32_t)kMaxDims; ++k)
      for (uint32_t e = (ok ? r.executed[k] : 0u) + lane; e < row_len; e += kBlock) {
        if (entry_bytes == 2) ((uint16_t*)rows)[k * row_len + e] = 0xFFFFu;
        else rows[k * row_len + e] = 0xFFu;
      }
  }
}

// ---------------------------------------------------------------------------
// themis_sweep (hot-path step a10): one lane per scenario x threshold x
// scheduler; the plan goes straight into LDS and only the time leaves.
// ---------------------------------------------------------------------------
template <bool kEager>
__device__ __forceinline__ void sweep_generic_evaluation(const Scenario& s, double chunk,
                                                         bool themis_on, bool rel, double th,
                                                         bool scf, uint64_t e, const Workspace& w,
                                                         const SimOut& out) {
  double load[kMaxDims];
#pragma unroll
  for (int k = 0; k < kMaxDims; ++k) load[k] = (k < s.D) ? tracker_start(s, k) : inf64();
  for (uint32_t c = 0; c < s.C; ++c) {
    uint32_t code = schedule_chunk(s, chunk, themis_on, rel, th, load);
    size_t at = (size_t)c * w.stride + e;
    w.meta[at] = code << 8;
    w.size[at] = chunk;
    w.arrival[at] = 0.0;
  }
  simulate_generic<kEager>(
      s, 1u, scf, w, e, [&](uint32_t) { return chunk; }, [&](uint32_t) { return 0.0; }, false,
      out);
}

// What one lane of a sweep evaluates.
struct SweepItem {
  uint64_t i;      // scenario
  double th;       // threshold
  bool themis_on;  // Themis or baseline order
  bool scf;        // Smallest-Chunk-First or FIFO
};

__device__ __forceinline__ SweepItem sweep_item(const themis_batch_t& b, uint64_t e, int n_thr,
                                                const double* thr, int thr_per_scenario,
                                                unsigned policy_mask, int n_pol) {
  SweepItem it;
  it.i = e / ((uint64_t)n_thr * n_pol);
  const uint32_t rem = (uint32_t)(e - it.i * (uint64_t)n_thr * n_pol);
  const int a = (int)(rem / (uint32_t)n_pol);
  const int col = (int)(rem - (uint32_t)a * (uint32_t)n_pol);
  // col-th set bit of the mask selects the scheduler
  int bit = 0;
  for (int seen = 0; bit < 3; ++bit)
    if (policy_mask & (1u << bit)) { if (seen == col) break; ++seen; }
  it.themis_on = bit != 0;
  it.scf = bit == 2;
  it.th = thr_per_scenario ? thr[(size_t)a * b.n + it.i] : thr[a];
  return it;
}

// The baseline order does not look at Alg. 1's threshold, so its column of a
// sweep needs one simulation per scenario, under the first threshold; the
// result is stored under every threshold.  A group of scenarios therefore has
// one workgroup per (threshold, scheduler) pair except the baseline's pairs
// beyond the first threshold: sweep_roles() of them.
__host__ __device__ __forceinline__ uint32_t sweep_roles(uint32_t n_thr, uint32_t n_pol,
                                                         unsigned policy_mask) {
  return n_thr * n_pol - ((policy_mask & THEMIS_SWEEP_BASELINE) ? n_thr - 1u : 0u);
}
// The pair a workgroup takes, as threshold * n_pol + column: the roles in turn,
// starting one further with every group (consecutive workgroups go to
// consecutive XCDs, and the number of roles is often a multiple of the eight
// XCDs: without the shift every XCD would see the same schedulers for every
// group, and they differ in cost).  Every workgroup of the grid has work, so
// the XCDs fill evenly -- workgroups are handed out in order, and a grid in
// which every eighth one returns at once keeps an eighth of the GPU idle.
__device__ __forceinline__ uint32_t sweep_block_role(uint32_t block, uint32_t n_thr, uint32_t n_pol,
                                                     unsigned policy_mask) {
  const uint32_t roles = sweep_roles(n_thr, n_pol, policy_mask);
  const uint32_t group = block / roles;
  const uint32_t r = (block - group * roles + group) % roles;
  if (!(policy_mask & THEMIS_SWEEP_BASELINE) || r < n_pol) return r;
  const uint32_t beyond = r - n_pol, others = n_pol - 1u;   // (others >= 1: r >= n_pol exists)
  return (1u + beyond / others) * n_pol + 1u + beyond % others;
}

// Stores the baseline's result under every threshold (NaN where that
// threshold itself is not valid).  e: the evaluation of the first threshold.
__device__ __forceinline__ void sweep_store_for_all_thresholds(
    const themis_batch_t& b, uint64_t i, uint64_t e, int n_thr, const double* thr,
    int thr_per_scenario, int n_pol, bool rel, double* t_done, double value,
    unsigned long long hand_over) {
  for (int a = 0; a < n_thr; ++a) {
    const double th = thr_per_scenario ? thr[(size_t)a * b.n + i] : thr[a];
    double* at = t_done + e + (uint64_t)a * (uint64_t)n_pol;
    if (!threshold_ok(th, rel)) *at = nan64();
    else if (hand_over) mark_left_to_generic(at, hand_over);
    else *at = value;
  }
}

// Thresholds that lead to the same plan.  Alg. 1 consults the threshold only to
// decide whether a chunk keeps the baseline order, so many thresholds of a
// study give a scenario the same plan (of eight between 0 and 1, four to five
// different ones on the networks measured), and a plan needs one simulation per
// queue policy.  sweep_plans_kernel finds, per scenario, which thresholds share
// a plan and lists one job for each of the different ones.
struct SweepJob {
  uint32_t i;      // scenario
  uint32_t same;   // the thresholds (one bit each) that give this plan
};
struct SweepJobs {
  const SweepJob* list;    // null: no list, every evaluation on its own
  const uint32_t* count;
};
constexpr uint32_t kSweepJobsMaxThr = 32;
constexpr size_t kSweepJobsHeader = 64;   // the counter
constexpr uint32_t kSweepPlansBlock = 8u * kBlock;

__global__ void sweep_clear_kernel(uint32_t* count) { *count = 0u; }

// One lane per (scenario, threshold), `width` lanes (a power of two) per
// scenario: all lanes of a scenario plan the same chunk at the same time, and
// after every chunk each compares its decision with the others'.  A plan is
// known by which of its chunks deviate from the baseline order: as long as two
// of them agree their loads are equal, and the order of the next chunk follows
// from the loads and that one decision.
// The places in the list are handed out by one counter, and an atomic on it
// takes some 13 ns however many wait.  With one per wavefront that was the time
// of the kernel on few chunks, so a workgroup is eight wavefronts (whole sweep,
// 65,536 scenarios, eight thresholds: 2-D, 4 chunks 158 -> 78 us, 16 chunks
// 309 -> 236 us; 4-D, 64 chunks 1,323 -> 1,279 us).
__global__ void __launch_bounds__(kSweepPlansBlock)
sweep_plans_kernel(themis_batch_t b, int n_thr, uint32_t width, const double* __restrict__ thr,
                   int thr_per_scenario, unsigned policy_mask, int n_pol, double* __restrict__ t_done,
                   SweepJob* __restrict__ list, uint32_t* __restrict__ count) {
  static_assert(kBlock == kPlanOrders, "one table entry per lane");
  __shared__ __attribute__((aligned(16))) uint32_t plan_orders[kPlanOrders * kPlanOrderWords];
  __shared__ uint32_t places[kSweepPlansBlock / kBlock];   // jobs of each wavefront, then where they go
  if (threadIdx.x < kPlanOrders) plan_order_entry(threadIdx.x, plan_orders + kPlanOrderWords * threadIdx.x);
  __syncthreads();
  const uint32_t lane = lane_id(), wave = threadIdx.x / kBlock, first = lane & ~(width - 1u);
  const uint32_t all = width == 32u ? ~0u : (1u << width) - 1u;
  const uint32_t a = lane - first;
  const uint64_t i = ((uint64_t)blockIdx.x * kSweepPlansBlock + threadIdx.x) / width;
  const bool exists = i < b.n && a < (uint32_t)n_thr;
  bool valid = false;
  uint32_t differ = 0u;
  if (i < b.n) {
    Scenario s = load_scenario(b, i);
    s.ctype = THEMIS_COLL_ALL_REDUCE;
    const bool rel = b.threshold_mode == THEMIS_THR_REL;
    const uint32_t at = exists ? a : 0u;
    const double th = thr_per_scenario ? thr[(size_t)at * b.n + i] : thr[at];
    const double S = b.size_bytes[i];
    if (s.valid && finite_positive(S)) {
      valid = exists && threshold_ok(th, rel);
      const uint32_t baseline = 0xe4u & ((1u << (2 * s.D)) - 1u);
      auto compare = [&](uint32_t, uint32_t code) {
        const bool off = code != baseline;
        const uint32_t others = (uint32_t)(__builtin_amdgcn_ballot_w64(off) >> first);
        differ |= off ? ~others : others;
      };
      const double chunk = S / (double)s.C;
      double load[kMaxDims];
      FastScenario fs;
      if (fast_eligible(s, chunk, THEMIS_MAX_CHUNKS, fs)) {
        plan_fast(s, fs, true, rel, th, load, compare, plan_orders);
      } else {
#pragma unroll
        for (int k = 0; k < kMaxDims; ++k) load[k] = (k < s.D) ? tracker_start(s, k) : inf64();
        for (uint32_t c = 0; c < s.C; ++c) compare(c, schedule_chunk(s, chunk, true, rel, th, load));
      }
    }
  }
  const uint32_t usable = (uint32_t)(__builtin_amdgcn_ballot_w64(valid) >> first) & all;
  const uint32_t same = ~differ & usable;
  const bool job = valid && (same & ((1u << a) - 1u)) == 0u;
  const uint64_t m = __builtin_amdgcn_ballot_w64(job);
  if (lane == 0u) places[wave] = (uint32_t)__builtin_popcountll(m);
  __syncthreads();
  if (threadIdx.x == 0u) {
    uint32_t sum = 0u;
    for (uint32_t w = 0; w < kSweepPlansBlock / kBlock; ++w) {
      const uint32_t jobs = places[w];
      places[w] = sum;
      sum += jobs;
    }
    const uint32_t base = sum != 0u ? atomicAdd(count, sum) : 0u;
    for (uint32_t w = 0; w < kSweepPlansBlock / kBlock; ++w) places[w] += base;
  }
  __syncthreads();
  if (job) {
    const uint32_t place = places[wave] + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                            __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    list[place] = SweepJob{(uint32_t)i, same};
  }
  if (exists && !valid)
    for (int p = (policy_mask & THEMIS_SWEEP_BASELINE) ? 1 : 0; p < n_pol; ++p)
      t_done[(i * (uint32_t)n_thr + a) * (uint32_t)n_pol + (uint32_t)p] = nan64();
}

// Where an evaluation's result goes.  With a list the evaluations are the
// baseline's (one per scenario, if it is asked for) and then every job under
// every Themis policy; the index of the first of its thresholds stands for a job.
struct SweepSlot {
  uint64_t e;       // index into t_done
  uint32_t same;    // the thresholds that share the result (0: only e itself)
  bool exists;
};
__device__ __forceinline__ SweepSlot sweep_job_slot(const SweepJobs& jobs, uint64_t j, uint32_t p, int n_thr,
                                                    unsigned policy_mask, int n_pol) {
  SweepSlot r;
  r.exists = j < *jobs.count;
  const SweepJob job = jobs.list[r.exists ? j : 0u];
  r.same = job.same;
  const uint32_t a = (uint32_t)__builtin_ctz(job.same | 0x80000000u);
  r.e = ((uint64_t)job.i * (uint32_t)n_thr + a) * (uint32_t)n_pol +
        ((policy_mask & THEMIS_SWEEP_BASELINE) ? 1u : 0u) + p;
  return r;
}
// kJobs as in sweep_kernel: the passes below are compiled apart for it, the
// choice at run time cost them 2 to 6 %.
template <bool kJobs>
__device__ __forceinline__ uint64_t sweep_evaluations(const themis_batch_t& b, const SweepJobs& jobs, int n_thr,
                                                      unsigned policy_mask, int n_pol) {
  if (!kJobs) return b.n * (uint64_t)n_thr * (uint64_t)n_pol;
  const bool base = (policy_mask & THEMIS_SWEEP_BASELINE) != 0u;
  return (base ? b.n : 0u) + (uint64_t)*jobs.count * (uint32_t)(n_pol - (base ? 1 : 0));
}
// (the baseline's result is first put under the first threshold that is valid)
__device__ __forceinline__ uint32_t sweep_first_valid(const themis_batch_t& b, uint64_t i, int n_thr,
                                                      const double* thr, int thr_per_scenario) {
  const bool rel = b.threshold_mode == THEMIS_THR_REL;
  for (int a = 0; a < n_thr; ++a)
    if (threshold_ok(thr_per_scenario ? thr[(size_t)a * b.n + i] : thr[a], rel)) return (uint32_t)a;
  return 0u;
}
template <bool kJobs>
__device__ __forceinline__ SweepSlot sweep_slot(const themis_batch_t& b, const SweepJobs& jobs, uint64_t x,
                                                int n_thr, const double* thr, int thr_per_scenario,
                                                unsigned policy_mask, int n_pol) {
  if (!kJobs) return SweepSlot{x, 0u, true};
  const bool base = (policy_mask & THEMIS_SWEEP_BASELINE) != 0u;
  const uint32_t per = (uint32_t)n_thr * (uint32_t)n_pol, themis = (uint32_t)(n_pol - (base ? 1 : 0));
  const uint64_t n_base = base ? b.n : 0u;
  if (x < n_base)
    return SweepSlot{x * per + sweep_first_valid(b, x, n_thr, thr, thr_per_scenario) * (uint32_t)n_pol, 0u, true};
  const uint64_t j = (x - n_base) / themis;
  return sweep_job_slot(jobs, j, (uint32_t)(x - n_base - j * themis), n_thr, policy_mask, n_pol);
}

// What the follow-up passes have put under the first of the thresholds that
// share a result goes to the others.
__global__ void __launch_bounds__(256)
sweep_spread_kernel(themis_batch_t b, SweepJobs jobs, int n_thr, const double* __restrict__ thr,
                    int thr_per_scenario, unsigned policy_mask, int n_pol, double* __restrict__ t_done,
                    unsigned long long call) {
  if (nothing_marked(call)) return;
  const uint64_t total = sweep_evaluations<true>(b, jobs, n_thr, policy_mask, n_pol);
  const uint64_t n_base = (policy_mask & THEMIS_SWEEP_BASELINE) ? b.n : 0u;
  for (uint64_t x = (uint64_t)blockIdx.x * 256u + threadIdx.x; x < total; x += (uint64_t)gridDim.x * 256u) {
    const SweepSlot slot = sweep_slot<true>(b, jobs, x, n_thr, thr, thr_per_scenario, policy_mask, n_pol);
    const double t = t_done[slot.e];
    if (x < n_base) {
      // (the others are marked as well where the follow-up passes had to come in)
      for (int a = 0; a < n_thr; ++a) {
        double* at = t_done + (x * (uint32_t)n_thr + (uint32_t)a) * (uint32_t)n_pol;
        if (is_left_to_generic(*at)) *at = t;
      }
      continue;
    }
    const uint32_t a = (uint32_t)__builtin_ctz(slot.same | 0x80000000u);
    for (uint32_t m = slot.same & (slot.same - 1u); m != 0u; m &= m - 1u)
      t_done[slot.e + (uint64_t)((uint32_t)__builtin_ctz(m) - a) * (uint32_t)n_pol] = t;
  }
}

// The evaluation a lane takes: `group` consecutive scenarios under one role per
// workgroup (`at`: the lane's place among them), or, from a list, `group` jobs
// under one Themis policy, behind the baseline's workgroups.
__device__ __forceinline__ SweepSlot sweep_lane_slot(const themis_batch_t& b, uint32_t workgroup, uint32_t group,
                                                     uint32_t at, int n_thr, unsigned policy_mask, int n_pol) {
  const uint32_t roles = sweep_roles((uint32_t)n_thr, (uint32_t)n_pol, policy_mask);
  const uint64_t i = (uint64_t)(workgroup / roles) * group + at;
  const bool exists = i < b.n;
  return SweepSlot{(exists ? i : 0u) * ((uint32_t)n_thr * (uint32_t)n_pol) +
                       sweep_block_role(workgroup, (uint32_t)n_thr, (uint32_t)n_pol, policy_mask),
                   0u, exists};
}
template <bool kBaseline>
__device__ __forceinline__ SweepSlot sweep_block_slot(const themis_batch_t& b, const SweepJobs& jobs,
                                                      uint32_t workgroup, uint32_t group, uint32_t at,
                                                      int n_thr, unsigned policy_mask, int n_pol) {
  const uint32_t base_blocks = kBaseline ? (uint32_t)((b.n + group - 1u) / group) : 0u;
  if (kBaseline && workgroup < base_blocks) {
    const uint64_t i = (uint64_t)workgroup * group + at;
    const bool exists = i < b.n;
    return SweepSlot{(exists ? i : 0u) * ((uint32_t)n_thr * (uint32_t)n_pol), 0u, exists};
  }
  const uint32_t block = workgroup - base_blocks, themis = (uint32_t)n_pol - (kBaseline ? 1u : 0u);
  const uint32_t g = block / themis;
  return sweep_job_slot(jobs, (uint64_t)g * group + at, block - g * themis, n_thr, policy_mask, n_pol);
}
template <bool kJobs>
__device__ __forceinline__ void sweep_store(const SweepSlot& slot, int n_pol, double* t_done, double value) {
  if (!kJobs) { t_done[slot.e] = value; return; }
  const uint32_t a = (uint32_t)__builtin_ctz(slot.same | 0x80000000u);
  for (uint32_t m = slot.same; m != 0u; m &= m - 1u)
    t_done[slot.e + (uint64_t)((uint32_t)__builtin_ctz(m) - a) * (uint32_t)n_pol] = value;
}

// kJobs: the evaluations come from a list (SweepJobs), after the baseline's.
// kBaseline: the sweep has a baseline column (compiled apart: what that
// column keeps alive across the event loop costs the other columns time).
template <typename L, bool kFix, bool kBaseline, bool kJobs>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(L::kWavesPerSimd)))
sweep_kernel(themis_batch_t b, int n_thr, const double* __restrict__ thr, int thr_per_scenario,
             unsigned policy_mask, int n_pol, double* __restrict__ t_done,
             unsigned long long hand_over, SweepJobs jobs) {
  __shared__ __attribute__((aligned(16))) uint32_t lds_block[L::kLaneWords * kBlock];
  // the planner's order table, in the place of the lists
  uint32_t* const plan_orders = lds_block + L::kPlanTableAt / 4u;
  plan_order_entry(threadIdx.x, plan_orders + kPlanOrderWords * threadIdx.x);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  // A wavefront takes 64 consecutive scenarios under one threshold and one
  // scheduler: its lanes read consecutive inputs, and on a batch that keeps to
  // one network they all take the same path through the event loop.
  const SweepSlot slot =
      kJobs ? sweep_block_slot<kBaseline>(b, jobs, blockIdx.x, kBlock, threadIdx.x, n_thr, policy_mask, n_pol)
            : sweep_lane_slot(b, blockIdx.x, kBlock, threadIdx.x, n_thr, policy_mask, n_pol);
  if (!slot.exists) return;
  const uint64_t e = slot.e;
  const SweepItem it = sweep_item(b, e, n_thr, thr, thr_per_scenario, policy_mask, n_pol);
  const bool every_threshold = kBaseline && !it.themis_on;   // (the same for the whole wavefront)

  Scenario s = load_scenario(b, it.i);
  s.ctype = THEMIS_COLL_ALL_REDUCE;  // sweeps evaluate All-Reduce only
  const bool rel = b.threshold_mode == THEMIS_THR_REL;
  const double S = b.size_bytes[it.i];
  const bool input_ok = s.valid && finite_positive(S);
  if (every_threshold) {
    if (!input_ok) {
      for (int a = 0; a < n_thr; ++a) t_done[e + (uint64_t)a * (uint64_t)n_pol] = nan64();
      return;
    }
  } else if (!(input_ok && threshold_ok(it.th, rel))) {
    t_done[e] = nan64();
    return;
  }

  const double chunk = S / (double)s.C;
  FastScenario fs;
  if (fast_eligible(s, chunk, L::kCap, fs)) {
    const LaneLds lds = lane_lds<L>(lds_block);
    double load[kMaxDims];
    plan_fast(s, fs, it.themis_on, rel, it.th, load,
              [&](uint32_t c, uint32_t code) { L::init_chunk(lds, c, code, 0u); }, plan_orders);
    // (every lane is through with the table before a list is in its place)
    __builtin_amdgcn_wave_barrier();
    FastOut fo;
    fo.queue_order = nullptr;
    fo.slots = b.max_chunks;
    // times only
    FastResult r =
        simulate_pow2<L, kNoQueueOrder, false, kFix>(s, Pow2Model(s, fs, it.scf), lds, fo);
    if (r.ok) {
      if (every_threshold)
        sweep_store_for_all_thresholds(b, it.i, e, n_thr, thr, thr_per_scenario, n_pol, rel, t_done,
                                       r.t_done, 0ull);
      else sweep_store<kJobs>(slot, n_pol, t_done, r.t_done);
      return;
    }
  }
  if (every_threshold)
    sweep_store_for_all_thresholds(b, it.i, e, n_thr, thr, thr_per_scenario, n_pol, rel, t_done,
                                   nan64(), hand_over);
  else if (hand_over) mark_left_to_generic(t_done + e, hand_over);
  else t_done[e] = nan64();
}

// The same with four lanes per evaluation (themis_quad.hpp): a wavefront takes
// 16 consecutive scenarios under one threshold and one scheduler.
template <uint32_t kChunks, bool kFix, bool kBaseline, bool kJobs>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(LayoutQuad<kChunks, 16>::kWavesPerSimd)))
sweep_quad_kernel(themis_batch_t b, int n_thr, const double* __restrict__ thr, int thr_per_scenario,
                  unsigned policy_mask, int n_pol, double* __restrict__ t_done,
                  unsigned long long hand_over, SweepJobs jobs) {
  using L = LayoutQuad<kChunks, 16>;
  __shared__ uint32_t lds_block[QuadPow2<L, kFix>::kBytes / 4u];
  const uint32_t quad = threadIdx.x >> 2;
  const SweepSlot slot =
      kJobs ? sweep_block_slot<kBaseline>(b, jobs, block_index(), L::kQuads, quad, n_thr, policy_mask, n_pol)
            : sweep_lane_slot(b, block_index(), L::kQuads, quad, n_thr, policy_mask, n_pol);
  if (__builtin_amdgcn_ballot_w64(slot.exists) == 0ull) return;   // (beyond the list, or the grid's last row)
  // a quad without an evaluation stays: the wavefront leaves the event loop as a whole
  const bool exists = slot.exists;
  const uint64_t e = exists ? slot.e : 0u;
  const SweepItem it = sweep_item(b, e, n_thr, thr, thr_per_scenario, policy_mask, n_pol);
  const bool writer = exists && (threadIdx.x & 3u) == 0u;   // one lane of the quad stores the result
  const bool every_threshold = kBaseline && !it.themis_on;   // (the same for the whole wavefront)

  Scenario s = load_scenario(b, it.i);
  s.ctype = THEMIS_COLL_ALL_REDUCE;  // sweeps evaluate All-Reduce only
  const bool rel = b.threshold_mode == THEMIS_THR_REL;
  const double S = b.size_bytes[it.i];
  const bool ok = s.valid && finite_positive(S) && (every_threshold || threshold_ok(it.th, rel));
  const double chunk = S / (double)s.C;
  FastScenario fs;
  const bool eligible = fast_eligible(s, chunk, L::kCap, fs);
  // (a quad without a valid scenario only keeps the others company: no chunks, no events)
  const bool fast = exists && ok && eligible;
  const uint32_t k = threadIdx.x & 3u;
  QuadQueue<L> queue(lds_block);
  if (fast)   // (a lane takes the chunks that start on its own dimension)
    plan_quad_pow2(s, fs, it.themis_on, rel, it.th, [&](uint32_t c, bool first, uint32_t order) {
      if (first) queue.add(c | (quad_row((uint32_t)s.D) + order) << 9);
    });
  const Pow2Model pow2(s, fs, it.scf);
  const QuadResult r = simulate_quad<L, false>(QuadPow2<L, kFix>(s, pow2, k, lds_block), queue, (uint32_t)pow2.ranktab & 15u,
                                               fast ? 2u * (uint32_t)s.D * s.C : 0u, pow2.t_min((uint32_t)s.D),
                                               [](uint32_t, uint32_t) {});
  if (!writer) return;
  if (every_threshold) {
    if (!ok) {
      for (int a = 0; a < n_thr; ++a) t_done[e + (uint64_t)a * (uint64_t)n_pol] = nan64();
    } else {
      const bool have = fast && r.ok;
      sweep_store_for_all_thresholds(b, it.i, e, n_thr, thr, thr_per_scenario, n_pol, rel, t_done,
                                     have ? r.t_done : nan64(), have ? 0ull : hand_over);
    }
    return;
  }
  if (!ok) t_done[e] = nan64();
  else if (fast && r.ok) sweep_store<kJobs>(slot, n_pol, t_done, r.t_done);
  else if (hand_over) mark_left_to_generic(t_done + e, hand_over);
  else t_done[e] = nan64();
}

// The same with a wavefront per evaluation (themis_wave.hpp): sweeps too small
// to fill the GPU otherwise.
template <uint32_t kWords>
__global__ void __launch_bounds__(kBlock)
sweep_wave_kernel(themis_batch_t b, int n_thr, const double* __restrict__ thr, int thr_per_scenario,
                  unsigned policy_mask, int n_pol, double* __restrict__ t_done,
                  unsigned long long hand_over) {
  __shared__ WaveLds<kWords> lds;
  __shared__ uint8_t codes[64u * kWords];
  const uint32_t lane = lane_id();
  const uint64_t e = sweep_lane_slot(b, blockIdx.x, 1u, 0u, n_thr, policy_mask, n_pol).e;
  const SweepItem it = sweep_item(b, e, n_thr, thr, thr_per_scenario, policy_mask, n_pol);
  const bool every_threshold = (policy_mask & THEMIS_SWEEP_BASELINE) != 0u && !it.themis_on;
  Scenario s = load_scenario(b, it.i);
  s.ctype = THEMIS_COLL_ALL_REDUCE;  // sweeps evaluate All-Reduce only
  const bool rel = b.threshold_mode == THEMIS_THR_REL;
  const double S = b.size_bytes[it.i];
  const bool input_ok = s.valid && finite_positive(S);
  double value = nan64();
  bool left = false;
  if (input_ok && (every_threshold || threshold_ok(it.th, rel))) {
    const double chunk = S / (double)s.C;
    double load[kMaxDims];
    wave_plan(s, chunk, it.themis_on, rel, it.th, load, [&](uint32_t first, uint32_t code) {
      codes[first + lane] = (uint8_t)code;
    });
    __syncthreads();
    WaveResult r;
    left = wave_simulate<kWords, false>(s, chunk, it.scf, lds, [&](uint32_t c) { return (uint32_t)codes[c]; }, r) !=
           WaveOutcome::kDone;
    value = r.t_done;
  }
  if (lane != 0u) return;
  if (every_threshold && input_ok)
    sweep_store_for_all_thresholds(b, it.i, e, n_thr, thr, thr_per_scenario, n_pol, rel, t_done, value,
                                   left ? hand_over : 0ull);
  else if (every_threshold)
    for (int a = 0; a < n_thr; ++a) t_done[e + (uint64_t)a * (uint64_t)n_pol] = nan64();
  else if (left) mark_left_to_generic(t_done + e, hand_over);
  else t_done[e] = value;
}

// The generic pass of themis_sweep: the evaluations still marked (kLdsSlots
// as in simulate_generic_pass).
template <uint32_t kLdsSlots, bool kJobs>
__device__ __forceinline__ void sweep_generic_pass(
    const themis_batch_t& b, int n_thr, const double* __restrict__ thr, int thr_per_scenario,
    unsigned policy_mask, int n_pol, double* __restrict__ t_done, const SweepJobs& jobs, Workspace w, void* lds_block) {
  if (kLdsSlots) w = carve_workspace(lds_block, kBlock, kLdsSlots);
  const uint64_t total = sweep_evaluations<kJobs>(b, jobs, n_thr, policy_mask, n_pol);
  const uint64_t groups = (total + kBlock - 1) / kBlock;
  for (uint64_t grp = blockIdx.x; grp < groups; grp += gridDim.x) {
    const uint64_t x = grp * kBlock + threadIdx.x;
    if (x >= total) continue;
    const uint64_t e = sweep_slot<kJobs>(b, jobs, x, n_thr, thr, thr_per_scenario, policy_mask, n_pol).e;
    if (!is_left_to_generic(t_done[e])) continue;
    const uint64_t col = kLdsSlots ? threadIdx.x : e;
    const SweepItem it = sweep_item(b, e, n_thr, thr, thr_per_scenario, policy_mask, n_pol);
    Scenario s = load_scenario(b, it.i);
    s.ctype = THEMIS_COLL_ALL_REDUCE;
    SimOut out;
    out.t_done = t_done + e;
    out.busy = nullptr;
    out.busy_stride = 0;
    out.queue_order = nullptr;
    out.entry_bytes = 1;
    out.slots = b.max_chunks;
    if (!kLdsSlots && !w.meta) { t_done[e] = nan64(); continue; }
    sweep_generic_evaluation<(kLdsSlots > 0)>(s, b.size_bytes[it.i] / (double)s.C, it.themis_on,
                                              b.threshold_mode == THEMIS_THR_REL, it.th, it.scf,
                                              col, w, out);
  }
}

template <uint32_t kLdsSlots, bool kJobs>
__global__ void __launch_bounds__(kBlock)
sweep_generic_kernel(themis_batch_t b, int n_thr, const double* __restrict__ thr,
                     int thr_per_scenario, unsigned policy_mask, int n_pol,
                     double* __restrict__ t_done, Workspace w, unsigned long long call, SweepJobs jobs) {
  __shared__ double lds_block[kLdsSlots ? generic_lds_bytes(kLdsSlots) / sizeof(double) : 1u];
  if (nothing_marked(call)) return;
  sweep_generic_pass<kLdsSlots, kJobs>(b, n_thr, thr, thr_per_scenario, policy_mask, n_pol, t_done, jobs, w,
                                lds_block);
}

// The same for themis_sweep: Alg. 1 with real divisions straight into the
// chunk words, then the table-driven event loop.
template <int kVariant, bool kJobs>
__device__ __forceinline__ void sweep_table_pass(
    const themis_batch_t& b, int n_thr, const double* __restrict__ thr, int thr_per_scenario,
    unsigned policy_mask, int n_pol, double* __restrict__ t_done, const SweepJobs& jobs, void* lds_block) {
  using L = typename TableVariant<kVariant>::L;
  constexpr bool kWide = kVariant != 0;
  const uint64_t total = sweep_evaluations<kJobs>(b, jobs, n_thr, policy_mask, n_pol);
  const uint64_t groups = (total + kBlock - 1) / kBlock;
  for (uint64_t grp = blockIdx.x; grp < groups; grp += gridDim.x) {
    const uint64_t x = grp * kBlock + threadIdx.x;
    if (x >= total) continue;
    const uint64_t e = sweep_slot<kJobs>(b, jobs, x, n_thr, thr, thr_per_scenario, policy_mask, n_pol).e;
    if (!is_left_to_generic(t_done[e])) continue;
    const SweepItem it = sweep_item(b, e, n_thr, thr, thr_per_scenario, policy_mask, n_pol);
    Scenario s = load_scenario(b, it.i);
    s.ctype = THEMIS_COLL_ALL_REDUCE;
    if (s.C > L::kCap) continue;
    const double chunk = b.size_bytes[it.i] / (double)s.C;
    const bool rel = b.threshold_mode == THEMIS_THR_REL;
    LaneLds lds;
    lds.base = (uint8_t*)lds_block + 4u * threadIdx.x;
    double load[kMaxDims];
#pragma unroll
    for (int k = 0; k < kMaxDims; ++k) load[k] = (k < s.D) ? tracker_start(s, k) : inf64();
    auto code_at = [&](uint32_t) { return schedule_chunk(s, chunk, it.themis_on, rel, it.th, load); };
    FastOut fo;
    fo.queue_order = nullptr;
    fo.slots = b.max_chunks;
    FastResult r;
    if constexpr (kVariant >= 3) {
      DivModelT<LayoutTableWide> model(s, lds, chunk, it.scf);
      table_setup_packed<L>(s, it.scf, lds, code_at, model);
      r = simulate_table_packed<L>(s, model, lds);
    } else if constexpr (kWide) {
      DivModelT<L> model(s, lds, chunk, it.scf);
      table_setup_wide<L>(s, it.scf, lds, code_at, model);
      r = simulate_fast<L, kNoQueueOrder, false, true>(s, model, lds, fo);
    } else {
      TableModel model;
      if (!table_setup(s, chunk, it.scf, lds, code_at, model)) continue;
      r = simulate_fast<L, kNoQueueOrder, false, true>(s, model, lds, fo);
    }
    if (r.ok) t_done[e] = r.t_done;
  }
}

// Everything that follows the LDS kernel of themis_sweep, in one launch (see
// simulate_follow_up_kernel).
template <int kTableA, int kTableB, uint32_t kGeneric, bool kJobs>
__global__ void __launch_bounds__(kBlock)
sweep_follow_up_kernel(themis_batch_t b, int n_thr, const double* __restrict__ thr,
                       int thr_per_scenario, unsigned policy_mask, int n_pol,
                       double* __restrict__ t_done, Workspace w, unsigned long long call, SweepJobs jobs) {
  constexpr size_t kBytes_ = max_bytes(max_bytes(table_lds_bytes<kTableA>(), table_lds_bytes<kTableB>()),
                                       kGeneric == kNoGeneric ? 0u : generic_lds_bytes(kGeneric));
  __shared__ double lds_block[kBytes_ ? (kBytes_ + 7u) / 8u : 1u];
  if (nothing_marked(call)) return;
  if constexpr (kTableA >= 0)
    sweep_table_pass<kTableA, kJobs>(b, n_thr, thr, thr_per_scenario, policy_mask, n_pol, t_done, jobs, lds_block);
  if constexpr (kTableB >= 0) {
    __syncthreads();
    sweep_table_pass<kTableB, kJobs>(b, n_thr, thr, thr_per_scenario, policy_mask, n_pol, t_done, jobs, lds_block);
  }
  if constexpr (kGeneric != kNoGeneric) {
    __syncthreads();
    sweep_generic_pass<kGeneric, kJobs>(b, n_thr, thr, thr_per_scenario, policy_mask, n_pol, t_done, jobs, w,
                                 lds_block);
  }
}

// ---------------------------------------------------------------------------
// themis_sweep_best: per scenario and scheduler the best threshold of a sweep
// and the speed-up over the baseline (Sec. 5.3, Sec. 6.1).  One lane per
// (scenario, scheduler).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
sweep_best_kernel(uint64_t n, uint32_t n_thr, uint32_t n_pol, const double* __restrict__ t_done,
                  int baseline_col, double* __restrict__ best_t, uint32_t* __restrict__ best_thr,
                  double* __restrict__ speedup) {
  const uint64_t e = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= n * n_pol) return;
  const uint64_t i = e / n_pol;
  const uint32_t p = (uint32_t)(e - i * n_pol);
  const double* row = t_done + i * n_thr * n_pol;
  double best = nan64();
  uint32_t at = 0xffffffffu;
  for (uint32_t a = 0; a < n_thr; ++a) {
    const double t = row[(size_t)a * n_pol + p];
    // the first value that is not NaN, then every strictly smaller one
    if (t == t && (at == 0xffffffffu || t < best)) { best = t; at = a; }
  }
  best_t[e] = best;
  if (best_thr) best_thr[e] = at;
  if (speedup && baseline_col >= 0) speedup[e] = row[baseline_col] / best;
}

// ---------------------------------------------------------------------------
// themis_search_batch: every assignment of dimension orders to chunks.
// ---------------------------------------------------------------------------
// (D!)^C if it does not exceed bound, else 0.
__device__ __forceinline__ uint64_t assignment_count(uint32_t D, uint32_t C, uint64_t bound) {
  const uint64_t F = factorial_u32(D);
  uint64_t total = 1;
  for (uint32_t c = 0; c < C; ++c) {
    if (total > bound / F) return 0;
    total *= F;
  }
  return total;
}

// A scenario's answer, NaN / all-ones if !ok (for one lane to write).
__device__ __forceinline__ void search_write(const themis_batch_t& b, uint64_t i, bool ok, double best,
                                             uint64_t arg, double* best_t, uint8_t* best_orders) {
  const uint32_t D = b.ndims[i], C = b.chunks[i];
  best_t[i] = ok ? best : nan64();
  if (!best_orders) return;
  uint8_t* out = best_orders + i * b.max_chunks;
  const uint32_t F = ok ? factorial_u32(D) : 1u;
  uint64_t rest = arg;
  for (uint32_t c = 0; c < b.max_chunks; ++c) {
    uint32_t code = 0xFFu;
    if (ok && c < C) {
      const uint64_t q = rest / F;
      code = nth_permutation_code(D, (uint32_t)(rest - q * F));
      rest = q;
    }
    out[c] = (uint8_t)code;
  }
}

// Smallest time of the wavefront and the lowest assignment number that reaches it, in lane 0.
__device__ __forceinline__ void search_lowest(double& best, uint64_t& arg) {
  for (int off = 32; off > 0; off >>= 1) {
    const double ob = __shfl_down(best, off);
    const uint64_t oa = ((uint64_t)__shfl_down((uint32_t)(arg >> 32), off) << 32) |
                        __shfl_down((uint32_t)arg, off);
    if (ob < best || (ob == best && oa < arg)) { best = ob; arg = oa; }
  }
}

// Up to kSearchFew assignments per scenario: too few lanes of a wavefront, and
// one simulation too short, for a table per scenario.  The first lane_blocks
// workgroups take what has power-of-two NPU counts, a lane per assignment and as
// many whole scenarios as fit 64 lanes; the others look for the rest in `group`
// scenarios each and simulate those on a shared table one by one (what that does
// not take goes the way of search_kernel's).  For batches of more scenarios than
// the GPU holds wavefronts; us, this / search_kernel, on power-of-two counts and on
// others: 2-D, 16,384 scenarios, 2 chunks 19 / 74 and 92 / 74, 4 chunks 53 / 105 and
// 136 / 105; 131,072, 4 chunks 294 / 750 and 951 / 755; 3-D, one chunk, 16,384
// 21 / 69 and 84 / 68; 4-D 51 / 84 and 314 / 300; 1-D, 64 chunks, 131,072 190 / 5,475.
// 64 assignments are as fast either way, 36 (one scenario in 64 lanes) 119 / 98.
constexpr uint32_t kSearchFew = 32u;
template <typename L, bool kFix>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(3)))
search_few_kernel(themis_batch_t b, uint32_t max_assign, uint32_t lane_blocks, uint32_t group,
                  double* __restrict__ times, double* __restrict__ best_t, uint8_t* __restrict__ best_orders,
                  unsigned long long call) {
  constexpr uint32_t kCap = L::kCap;
  constexpr uint32_t kRingBytes = kCap * 128u + LayoutRing::kTailBytes;
  struct Shared { uint8_t ring[kRingBytes]; SharedTable tab; };
  __shared__ union Block {
    uint32_t lanes[L::kLaneWords * kBlock];
    __attribute__((aligned(16))) Shared shared;
    __device__ Block() {}
  } block;
  const uint32_t lane = threadIdx.x;
  FastOut none;
  none.queue_order = nullptr;
  none.slots = b.max_chunks;
  auto count_of = [&](const Scenario& s, double S) {
    return s.valid && finite_positive(S) && s.C <= kCap
               ? (uint32_t)assignment_count((uint32_t)s.D, s.C, (uint64_t)max_assign) : 0u;
  };

  if (blockIdx.x < lane_blocks) {
    const uint32_t per = kBlock / max_assign, seg = lane / max_assign, a = lane - seg * max_assign;
    const uint64_t i = (uint64_t)blockIdx.x * per + seg;
    const bool exists = seg < per && i < b.n;
    double best = inf64();
    uint32_t arg = a;
    bool bad = false, answer = false;   // whether the scenario's answer is given here
    if (exists) {
      const Scenario s = load_scenario(b, i);
      const double S = b.size_bytes[i], chunk = S / (double)s.C;
      const uint32_t count = count_of(s, S);
      FastScenario fs;
      answer = count == 0u || fast_eligible(s, chunk, kCap, fs);
      bad = count == 0u;
      if (answer && a < count) {
        const LaneLds lds = lane_lds<L>(block.lanes);
        const DivideByOrders by_orders((uint32_t)s.D);
        const uint32_t F = factorial_u32((uint32_t)s.D);
        uint32_t rest = a;
        for (uint32_t c = 0; c < s.C; ++c) {
          const uint32_t q = by_orders(rest);
          L::init_chunk(lds, c, stored_code(s, fs, nth_permutation_code((uint32_t)s.D, rest - q * F)), fs.state0);
          rest = q;
        }
        const FastResult r = simulate_pow2<L, kNoQueueOrder, false, kFix>(
            s, Pow2Model(s, fs, b.intra_policy[i] == THEMIS_INTRA_SCF), lds, none);
        bad = !r.ok;
        if (r.ok) best = r.t_done;
      }
    }
    const uint64_t gave_up = __builtin_amdgcn_ballot_w64(bad);
    for (uint32_t off = 32u; off > 0u; off >>= 1) {   // (the scenario's lanes only)
      const double ob = __shfl_down(best, off);
      const uint32_t oa = (uint32_t)__shfl_down((int)arg, off);
      if (a + off < max_assign && (ob < best || (ob == best && oa < arg))) { best = ob; arg = oa; }
    }
    const uint64_t mine = ((1ull << max_assign) - 1ull) << (lane & 63u);   // (of lane a == 0)
    if (answer && a == 0u) search_write(b, i, (gave_up & mine) == 0ull, best, arg, best_t, best_orders);
    return;
  }

  // (which of the group they are: a lane each)
  const uint64_t first = (uint64_t)(blockIdx.x - lane_blocks) * group;
  bool other = false;
  if (lane < group && first + lane < b.n) {
    const Scenario s = load_scenario(b, first + lane);
    const double S = b.size_bytes[first + lane];
    FastScenario fs;
    other = count_of(s, S) != 0u && !fast_eligible(s, S / (double)s.C, kCap, fs);
  }
  for (uint64_t left = __builtin_amdgcn_ballot_w64(other); left != 0ull; left &= left - 1ull) {
    const uint64_t i = first + (uint32_t)__builtin_ctzll(left);
    const Scenario s = load_scenario(b, i);
    const double S = b.size_bytes[i];
    const uint32_t count = count_of(s, S);
    const SharedSetup setup = shared_table<false>(s, S / (double)s.C, b.intra_policy[i] == THEMIS_INTRA_SCF,
                                           block.shared.tab);
    __syncthreads();
    if (!setup.ok) {
      if (lane < max_assign) times[i * max_assign + lane] = lane < count ? left_to_generic() : inf64();
      if (lane == 0u) mark_left_to_generic(best_t + i, call);
      __syncthreads();
      continue;
    }
    double best = inf64();
    uint64_t arg = ~0ull;
    bool bad = false;
    if (lane < count) {
      const DivideByOrders by_orders((uint32_t)s.D);
      const uint32_t F = factorial_u32((uint32_t)s.D);
      LaneLds lds;
      lds.base = block.shared.ring + LayoutRing::lane_term_rec(lane);
      lds.aux = block.shared.ring + kCap * 128u + (LayoutRing::lane_term_tail(lane) - LayoutRing::kRecBytes);
      uint32_t rest = lane;
      auto rank_at = [&](uint32_t) {
        const uint32_t q = by_orders(rest), digit = rest - q * F;
        rest = q;
        return (uint32_t)block.shared.tab.rank_of[digit];
      };
      const SharedModel model(block.shared.tab, setup, s.ctype, rank_at);
      const FastResult r = shared_ring<false>(s, model, lds);
      bad = !r.ok;
      if (r.ok) { best = r.t_done; arg = lane; }
    }
    bad = __builtin_amdgcn_ballot_w64(bad) != 0ull;
    search_lowest(best, arg);
    if (lane == 0u) search_write(b, i, !bad, best, arg, best_t, best_orders);
    __syncthreads();
  }
}

// `parts` wavefronts per scenario, each with every parts-th group of 64
// assignments.  An assignment whose lower bound (SharedBound) is above a time
// already found cannot be the answer, so only the others are simulated: first
// the one with the lowest bound of every lane, which puts the limit close to
// the answer, then what is still below it, gathered 64 at a time so that the
// lanes of a simulation are full.  On three dimensions and four chunks that
// leaves 100 of 1,296 assignments (simulating all of them: 3.1 ms for 16,384
// scenarios, against the limit 0.5 ms).  Where a schedule could take so long that its
// shortest stage no longer moves the clock nothing is left out, so that the
// scenario is found to be out of range.
// kCap: chunk records in LDS; Index: type of an assignment number.
// Scenarios the shared table does not take (more than 16 size classes, sizes
// outside the normal range) are marked and go through search_table_kernel and
// search_finish_kernel.
template <uint32_t kCap, typename Index>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(3)))
search_kernel(themis_batch_t b, uint64_t max_assign, uint32_t parts, double* __restrict__ times,
              double* __restrict__ best_t, uint8_t* __restrict__ best_orders, unsigned long long call) {
  __shared__ __attribute__((aligned(16))) uint8_t ring[kCap * 128u + LayoutRing::kTailBytes];
  __shared__ SharedTable tab;
  __shared__ Index queue[2u * kBlock];
  const uint64_t i = blockIdx.x / parts;
  const uint32_t part = (uint32_t)(blockIdx.x - i * parts), lane = threadIdx.x;
  Scenario s = load_scenario(b, i);
  const bool scf = b.intra_policy[i] == THEMIS_INTRA_SCF;
  const double S = b.size_bytes[i];
  const bool valid = s.valid && finite_positive(S) && s.C <= kCap;
  const uint64_t all = valid ? assignment_count((uint32_t)s.D, s.C, max_assign) : 0u;
  double* row = times + i * max_assign;
  // what this wavefront found: the answer itself, or its part of it
  auto report = [&](bool ok, double best, uint64_t arg) {
    if (lane != 0u) return;
    if (parts == 1u) { search_write(b, i, ok, best, arg, best_t, best_orders); return; }
    row[part] = ok ? best : nan64();
    ((uint64_t*)row)[parts + part] = arg;
    if (part == 0u) best_t[i] = 0.0;   // (whatever it held: not a mark)
  };
  if (all == 0u) { report(false, nan64(), 0u); return; }
  const Index count = (Index)all;
  const double chunk = S / (double)s.C;
  const SharedSetup setup = shared_table<false>(s, chunk, scf, tab);
  __syncthreads();
  if (!setup.ok) {
    for (uint64_t a = (uint64_t)part * kBlock + lane; a < max_assign; a += (uint64_t)parts * kBlock)
      row[a] = a < all ? left_to_generic() : inf64();
    if (part == 0u && lane == 0u) mark_left_to_generic(best_t + i, call);
    return;
  }
  const double longest = (double)s.C * setup.t_max * (1.0 + 1e-9);
  // (nor where single precision does not resolve the times)
  const bool prune = longest + 0.25 * setup.t_min > longest && longest < inf64() && setup.t_min > 1e-30;

  const uint32_t D = (uint32_t)s.D, C = s.C, F = factorial_u32(D);
  const bool both = s.ctype == THEMIS_COLL_ALL_REDUCE;
  const DivideByOrders by_orders(D);
  auto bound = [&](Index a) {
    SharedBound lb;
    for (uint32_t c = 0; c < C; ++c) {
      const Index q = by_orders(a);
      lb.add(tab, tab.rank_of[(uint32_t)(a - q * (Index)F)], both);
      a = q;
    }
    return lb.value(both);
  };
  LaneLds lds;
  lds.base = ring + LayoutRing::lane_term_rec(lane);
  lds.aux = ring + kCap * 128u + (LayoutRing::lane_term_tail(lane) - LayoutRing::kRecBytes);

  const Index first = (Index)part * kBlock, step = (Index)parts * kBlock;
  // (one group per wavefront: all of it at once, no bounds)
  const bool one_group = count <= step;
  Index seed = first + lane;
  bool seeded = one_group && seed < count;
  if (!one_group) {
    float lowest = 0.0f;
    for (Index from = first; from < count; from += step) {
      const Index a = from + lane;
      if (a < count) {
        const float lb = bound(a);
        if (!seeded || lb < lowest) { lowest = lb; seed = a; seeded = true; }
      }
      if (count - from <= step) break;   // (no wrap of the index)
    }
  }
  double best = inf64(), limit = inf64();
  uint64_t arg = ~0ull;
  bool bad = false, first_round = true, scanned = one_group || first >= count;
  Index from = first;
  uint32_t queued = 0u;
  for (;;) {
    Index a = seed;
    bool active = seeded;
    if (!first_round) {
      const float above = (float)limit * (1.0f + 1e-6f);
      while (queued < kBlock && !scanned) {
        const Index x = from + lane;
        const bool take = x < count && x != seed && !(prune && bound(x) > above);
        const uint64_t m = __builtin_amdgcn_ballot_w64(take);
        if (take)
          queue[queued + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] = x;
        queued += (uint32_t)__builtin_popcountll(m);
        scanned = count - from <= step;
        from += step;
      }
      if (queued == 0u) break;
      __syncthreads();
      active = lane < queued;
      a = queue[lane];
      const Index rest = queue[kBlock + lane];
      __syncthreads();
      queue[lane] = rest;
      queued = queued > kBlock ? queued - kBlock : 0u;
    }
    first_round = false;
    if (active) {
      Index rest = a;
      auto rank_at = [&](uint32_t) {
        const Index q = by_orders(rest);
        const uint32_t digit = (uint32_t)(rest - q * (Index)F);
        rest = q;
        return (uint32_t)tab.rank_of[digit];
      };
      const SharedModel model(tab, setup, s.ctype, rank_at);
      const FastResult r = shared_ring<false>(s, model, lds);
      bad = bad || !r.ok;
      if (r.ok && (r.t_done < best || (r.t_done == best && a < arg))) { best = r.t_done; arg = a; }
    }
    double lowest = best;
    for (int off = 32; off > 0; off >>= 1) lowest = min_f64(lowest, __shfl_xor(lowest, off));
    limit = lowest;
  }
  bad = __builtin_amdgcn_ballot_w64(bad) != 0ull;
  search_lowest(best, arg);
  report(!bad, best, arg);
}

// The scenarios that search_kernel has marked, on per-order tables of their own
// in every lane: one lane per (scenario, assignment), times[i * max_assign + a].
// Strides over all slots with a grid that just fills the device and returns at
// once if nothing is marked (see g_marked_call).
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(LayoutTableWide::kWavesPerSimd)))
search_table_kernel(themis_batch_t b, uint64_t max_assign, double* __restrict__ times,
                    const double* __restrict__ best_t, unsigned long long call) {
  using L = LayoutTableWide;
  __shared__ uint32_t lds_block[L::kLaneWords * kBlock];
  if (nothing_marked(call)) return;
  const uint64_t total = b.n * max_assign;
  for (uint64_t e = (uint64_t)blockIdx.x * kBlock + threadIdx.x; e < total;
       e += (uint64_t)gridDim.x * kBlock) {
    const uint64_t i = e / max_assign;
    const uint64_t a = e - i * max_assign;
    // (search_kernel writes all of a row only where it leaves the scenario; the
    // others hold whatever the caller's memory held, a mark's bits for instance)
    if (!is_left_to_generic(best_t[i]) || !is_left_to_generic(times[e])) continue;
    Scenario s = load_scenario(b, i);
    const bool scf = b.intra_policy[i] == THEMIS_INTRA_SCF;
    const double chunk = b.size_bytes[i] / (double)s.C;
    const uint32_t F = factorial_u32((uint32_t)s.D);
    // digit c of the assignment number, base D!
    auto code_at = [&](uint32_t c) {
      uint64_t rest = a;
      for (uint32_t j = 0; j < c; ++j) rest /= F;
      return nth_permutation_code((uint32_t)s.D, (uint32_t)(rest % F));
    };
    FastOut fo;
    fo.queue_order = nullptr;
    fo.slots = b.max_chunks;
    LaneLds lds;
    lds.base = (uint8_t*)lds_block + 4u * threadIdx.x;
    DivModelT<L> model(s, lds, chunk, scf);
    table_setup_wide<L>(s, scf, lds, code_at, model);
    const FastResult r = simulate_fast<L, kNoQueueOrder, false, true>(s, model, lds, fo);
    times[e] = r.ok ? r.t_done : nan64();
  }
}

// What is left to do per scenario: the smallest of the times of a marked one,
// or of the parts it was searched in.
__global__ void __launch_bounds__(kBlock)
search_finish_kernel(themis_batch_t b, uint64_t max_assign, uint32_t parts,
                     const double* __restrict__ times, double* __restrict__ best_t,
                     uint8_t* __restrict__ best_orders, unsigned long long call) {
  if (parts == 1u && nothing_marked(call)) return;
  for (uint64_t i = blockIdx.x; i < b.n; i += gridDim.x) {
    const double* row = times + i * max_assign;
    double best = inf64();
    uint64_t arg = ~0ull;
    bool bad = false;
    if (is_left_to_generic(best_t[i])) {
      for (uint64_t a = threadIdx.x; a < max_assign; a += kBlock) {
        const double t = row[a];
        bad |= !(t == t);
        if (t < best) { best = t; arg = a; }  // ascending a per lane: the first minimum stays
      }
    } else if (parts > 1u) {
      for (uint32_t p = threadIdx.x; p < parts; p += kBlock) {
        const double t = row[p];
        const uint64_t a = ((const uint64_t*)row)[parts + p];
        bad |= !(t == t);
        if (t < best || (t == best && a < arg)) { best = t; arg = a; }
      }
    } else {
      continue;
    }
    bad = __builtin_amdgcn_ballot_w64(bad) != 0ull;
    search_lowest(best, arg);
    if (threadIdx.x == 0u) search_write(b, i, !bad && arg != ~0ull, best, arg, best_t, best_orders);
  }
}

// ---------------------------------------------------------------------------
// themis_beam_search_batch: the chunks get their orders one after the other,
// and after every chunk the `width` best partial schedules are kept (Sec. 4.1,
// observation 2, names the space; Alg. 1 walks it keeping one).
// ---------------------------------------------------------------------------
constexpr uint32_t kBeamMaxWidth = 64;
constexpr uint32_t kBeamOrders = 24;  // D! <= 24 candidates per kept schedule

// One scenario's part of the workspace is found through these offsets.
struct BeamLayout {
  uint64_t n;
  uint32_t width, mc;
  size_t off_digits[2], off_rank[2], off_live, off_times, off_best, off_greedy_orders,
      off_greedy_t, bytes;
};
__host__ __device__ inline BeamLayout beam_layout(uint64_t n, uint32_t mc, uint32_t width) {
  BeamLayout l;
  l.n = n; l.width = width; l.mc = mc;
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o = (o + bytes + 63u) & ~(size_t)63u; return at; };
  l.off_times = take((size_t)n * width * kBeamOrders * sizeof(double));
  l.off_best = take((size_t)n * sizeof(double));
  l.off_greedy_t = take((size_t)n * sizeof(double));
  l.off_live = take((size_t)n * sizeof(uint32_t));
  for (int h = 0; h < 2; ++h) {
    l.off_digits[h] = take((size_t)n * width * mc);
    l.off_rank[h] = take((size_t)n * width);
  }
  l.off_greedy_orders = take((size_t)n * mc);
  l.bytes = o;
  return l;
}

// Collective of the first m chunks of a C-chunk schedule: m chunks of size / m bytes.
__device__ __forceinline__ double beam_partial_size(double S, uint32_t C, uint32_t m) {
  return m == C ? S : (S / (double)C) * (double)m;
}

__global__ void __launch_bounds__(256)
beam_init_kernel(themis_batch_t b, BeamLayout l, uint8_t* __restrict__ ws) {
  const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= b.n) return;
  const Scenario s = load_scenario(b, i);
  const bool ok = s.valid && finite_positive(b.size_bytes[i]) && s.C <= 64u;
  ((uint32_t*)(ws + l.off_live))[i] = ok ? 1u : 0u;   // the empty schedule
  (ws + l.off_rank[0])[i * l.width] = 0u;
}

// One lane per (scenario, kept schedule, order of chunk m - 1): its time into
// times[i][p * 24 + j], +inf where there is no such candidate, NaN where the
// simulation gave up.  kTable: the scenarios the power-of-two path does not
// take (other NPU counts), on per-order tables; each kernel leaves the other's
// scenarios alone.  kLeft: the scenarios that beam_kernel of call
// left_by has left open (all of them go on the tables).
template <bool kTable, bool kFix, bool kLeft>
__global__ void __launch_bounds__(kBlock)
    __attribute__((amdgpu_waves_per_eu(kTable ? LayoutTableWide::kWavesPerSimd : LayoutRing::kWavesPerSimd)))
beam_eval_kernel(themis_batch_t b, BeamLayout l, uint8_t* __restrict__ ws, uint32_t m, int half,
                 unsigned long long left_by) {
  using L = typename std::conditional<kTable, LayoutTableWide, LayoutRing>::type;
  __shared__ uint32_t lds_block[L::kLaneWords * kBlock];
  if (kLeft && nothing_marked(left_by)) return;
  const uint64_t e = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  const uint32_t per = l.width * kBeamOrders;
  if (e >= b.n * per) return;
  const uint64_t i = e / per;
  const uint32_t cand = (uint32_t)(e - i * per);
  const uint32_t p = cand / kBeamOrders, j = cand - p * kBeamOrders;
  double* times = (double*)(ws + l.off_times);
  Scenario s = load_scenario(b, i);
  const uint32_t live = ((const uint32_t*)(ws + l.off_live))[i];
  const uint32_t C = s.C;
  if (live == 0u || (kLeft && live > kBeamMaxWidth) || m > C) return;       // nothing to do for this scenario
  const uint32_t F = factorial_u32((uint32_t)s.D);
  const double chunk = beam_partial_size(b.size_bytes[i], C, m) / (double)m;
  s.C = m;
  FastScenario fs;
  const bool pow2 = fast_eligible(s, chunk, LayoutRing::kCap, fs);
  if (!kLeft && pow2 == kTable) return;         // the other kernel's scenario
  if (p >= live || j >= F) { times[e] = inf64(); return; }
  const bool scf = b.intra_policy[i] == THEMIS_INTRA_SCF;
  const uint8_t* digits = ws + l.off_digits[half] + (i * l.width + p) * l.mc;
  auto code_at = [&](uint32_t c) {
    return nth_permutation_code((uint32_t)s.D, c + 1u == m ? j : (uint32_t)digits[c]);
  };
  FastOut fo;
  fo.queue_order = nullptr;
  fo.slots = b.max_chunks;
  FastResult r;
  if constexpr (kTable) {
    LaneLds lds;
    lds.base = (uint8_t*)lds_block + 4u * threadIdx.x;
    DivModelT<L> model(s, lds, chunk, scf);
    table_setup_wide<L>(s, scf, lds, code_at, model);
    r = simulate_fast<L, kNoQueueOrder, false, true>(s, model, lds, fo);
  } else {
    const LaneLds lds = lane_lds<L>(lds_block);
    for (uint32_t c = 0; c < m; ++c) L::init_chunk(lds, c, stored_code(s, fs, code_at(c)), fs.state0);
    r = simulate_pow2<L, kNoQueueOrder, false, kFix>(s, Pow2Model(s, fs, scf), lds, fo);
  }
  times[e] = r.ok ? r.t_done : nan64();
}

// One wavefront per scenario keeps the `width` best candidates: smaller time
// first, equal times in ascending assignment number (the newest chunk's digit
// is the most significant, then the kept schedule's own number, known by its
// rank among the kept ones).
template <bool kLeft>
__global__ void __launch_bounds__(kBlock)
beam_select_kernel(themis_batch_t b, BeamLayout l, uint8_t* __restrict__ ws, uint32_t m, int half,
                   unsigned long long left_by) {
  __shared__ uint32_t new_key[kBeamMaxWidth];
  if (kLeft && nothing_marked(left_by)) return;
  const uint64_t i = blockIdx.x;
  uint32_t* live_p = (uint32_t*)(ws + l.off_live) + i;
  const uint32_t live = *live_p;
  const uint32_t D = b.ndims[i], C = b.chunks[i];
  if (live == 0u || (kLeft && live > kBeamMaxWidth) || m > C) return;
  const uint32_t F = factorial_u32(D);
  const double* times = (const double*)(ws + l.off_times) + i * l.width * kBeamOrders;
  const uint8_t* rank_in = ws + l.off_rank[half] + i * l.width;
  uint8_t* rank_out = ws + l.off_rank[half ^ 1] + i * l.width;
  const uint8_t* digits_in = ws + l.off_digits[half] + i * l.width * l.mc;
  uint8_t* digits_out = ws + l.off_digits[half ^ 1] + i * l.width * l.mc;
  const uint32_t nc = live * F;
  const uint32_t kept = nc < l.width ? nc : l.width;
  bool bad = false;
  for (uint32_t x = threadIdx.x; x < nc; x += kBlock) {
    const uint32_t px = x / F, jx = x - px * F;
    const double tx = times[px * kBeamOrders + jx];
    bad |= !(tx == tx);
    const uint32_t kx = jx * kBeamMaxWidth + rank_in[px];
    uint32_t before = 0;
    for (uint32_t y = 0; y < nc; ++y) {
      const uint32_t py = y / F, jy = y - py * F;
      const double ty = times[py * kBeamOrders + jy];
      const uint32_t ky = jy * kBeamMaxWidth + rank_in[py];
      before += (ty < tx || (ty == tx && ky < kx)) ? 1u : 0u;
    }
    if (before < kept) {
      uint8_t* row = digits_out + before * l.mc;
      for (uint32_t c = 0; c + 1u < m; ++c) row[c] = digits_in[px * l.mc + c];
      row[m - 1u] = (uint8_t)jx;
      new_key[before] = kx;
      if (before == 0u) ((double*)(ws + l.off_best))[i] = tx;
    }
  }
  const bool any_bad = __syncthreads_or(bad ? 1 : 0) != 0;
  if (threadIdx.x < kept) {
    uint32_t smaller = 0;
    for (uint32_t q = 0; q < kept; ++q) smaller += new_key[q] < new_key[threadIdx.x] ? 1u : 0u;
    rank_out[threadIdx.x] = (uint8_t)smaller;
  }
  // a simulation that gave up: the scenario has no answer
  if (threadIdx.x == 0) *live_p = any_bad ? 0u : kept;
}

// One wavefront per scenario takes the whole beam search of it: per chunk slot m
// it makes the candidates (kept schedule x order of chunk m - 1), simulates
// them a lane each on a stage table that all lanes share, and keeps the best.
// With a lane per candidate of the whole batch and a selection kernel between
// the steps (above), every candidate is simulated, kept schedules and times go
// through HBM once per step, and other NPU counts take 60 KiB of LDS per wavefront.
// 4,096 scenarios: 4-D, width 4, 64 chunks 33.6 -> 29.8 ms; 2-D, width 8, 32
// chunks 14.8 -> 5.2 ms; of mixed dimensions, width 8, 24 chunks 13.9 -> 10.2 ms.
// Around the simulations nothing waits for LDS one value at a time (the first
// lists are linked in registers, selections halve over registers, lanes share a
// kept schedule's sums), and the stage table is made anew only where the chunk
// size has changed: 29.6 -> 25.6 ms.
//
// What bounds a step is the chain of events of a simulation round, so it should
// take one: where there are more candidates than lanes, those with the lowest
// bounds of their time (SharedBound) go first, and then only what could still
// be among the `width` best (a third of the candidates on the bench networks
// at width 4).  Nothing is left out where a stage might not move the clock, so
// that such a scenario is found to be out of range, and where single precision
// does not resolve the times.
//
// A candidate is kept * D! + order; smaller time first, equal times in
// ascending assignment number (the newest chunk's digit is the most
// significant, then the kept schedule's own number, known by its rank among
// the kept ones).
// Scenarios the shared table does not take (more than 16 size classes, as four
// dimensions of other NPU counts have, or sizes outside the normal range) are
// left to the step-wise kernels above.
constexpr uint32_t kBeamDone = 0x80000000u;   // (live of a scenario with an answer)

template <uint32_t kWidth>
struct BeamLds {
  static constexpr uint32_t kMost = kWidth * kBeamOrders;
  double time[kMost];
  uint32_t lb[kMost];          // bits of the bound (positive single precision); all ones: simulated
  uint32_t tb[kMost];          // bits of the time, rounded up; all ones: not simulated
  float4 prefix_of[kWidth][(sizeof(SharedBound) + 15u) / 16u];  // the kept schedules' SharedBound
  uint16_t list[kMost];
  uint16_t key[kWidth];        // order * 64 + rank of the kept schedule's parent
  uint8_t parent[kWidth], rank[kWidth];
  __attribute__((aligned(4))) uint8_t orders[2][kWidth][64];   // the kept schedules: a chunk's order rank
  __device__ __forceinline__ SharedBound& prefix(uint32_t p) { return *(SharedBound*)prefix_of[p]; }
};

// Smallest value that at least k of the n values do not exceed (all ones if there are fewer).
// The values stay in registers over the 32 halvings (kMost: the most there can be).
template <uint32_t kMost>
__device__ __forceinline__ uint32_t beam_kth(const uint32_t* v, uint32_t n, uint32_t k) {
  constexpr uint32_t kRegs = (kMost + kBlock - 1u) / kBlock;
  uint32_t mine[kRegs];
#pragma unroll
  for (uint32_t r = 0; r < kRegs; ++r) {
    const uint32_t x = r * kBlock + threadIdx.x;
    mine[r] = x < n ? v[x] : ~0u;   // (never counted: the middle is below all ones)
  }
  uint32_t lo = 0u, hi = ~0u;
  while (lo < hi) {
    const uint32_t mid = lo + (hi - lo) / 2u;
    uint32_t count = 0u;
#pragma unroll
    for (uint32_t r = 0; r < kRegs; ++r) {
      if (kRegs <= 2u || r * kBlock < n)
        count += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(mine[r] <= mid));
    }
    if (count >= k) hi = mid; else lo = mid + 1u;
  }
  return lo;
}
// The places of the values not above `most`, in ascending order, up to `room` of them.
__device__ __forceinline__ uint32_t beam_gather(const uint32_t* v, uint32_t n, uint32_t most, uint32_t room,
                                                uint16_t* list) {
  uint32_t got = 0u;
  for (uint32_t from = 0; from < n && got < room; from += kBlock) {
    const uint32_t x = from + threadIdx.x;
    const bool take = x < n && v[x < n ? x : 0u] <= most;
    const uint64_t set = __builtin_amdgcn_ballot_w64(take);
    const uint32_t at = got + __builtin_amdgcn_mbcnt_hi((uint32_t)(set >> 32),
                                                        __builtin_amdgcn_mbcnt_lo((uint32_t)set, 0u));
    if (take && at < room) list[at] = (uint16_t)x;
    got += (uint32_t)__builtin_popcountll(set);
  }
  return got < room ? got : room;
}

template <uint32_t kWidth>
__global__ void __launch_bounds__(kBlock)
    __attribute__((amdgpu_waves_per_eu(kWidth <= 4u ? 3 : kWidth <= 16u ? 2 : 1)))
beam_kernel(themis_batch_t b, BeamLayout l, uint8_t* __restrict__ ws, unsigned long long call) {
  constexpr uint32_t kCap = LayoutRing::kCap, kMost = BeamLds<kWidth>::kMost;
  __shared__ __attribute__((aligned(16))) uint8_t block[kCap * 128u + LayoutRing::kTailBytes];
  __shared__ SharedTable tab;
  __shared__ BeamLds<kWidth> k;
  const uint64_t i = blockIdx.x;
  const uint32_t lane = threadIdx.x;
  uint32_t* live_p = (uint32_t*)(ws + l.off_live) + i;
  Scenario s = load_scenario(b, i);
  const bool scf = b.intra_policy[i] == THEMIS_INTRA_SCF;
  const double S = b.size_bytes[i];
  if (!s.valid || !finite_positive(S) || s.C > kCap) {
    if (lane == 0u) *live_p = 0u;
    return;
  }
  const uint32_t D = (uint32_t)s.D, C = s.C, F = factorial_u32(D);
  const bool both = s.ctype == THEMIS_COLL_ALL_REDUCE;
  const DivideByOrders by_orders(D);
  SharedSetup setup;
  double made_for = -1.0;   // chunk size of the table
  uint32_t live = 1u;   // the empty schedule
  if (lane == 0u) k.rank[0] = 0u;
  for (uint32_t m = 1; m <= C; ++m) {
    const uint32_t half = m & 1u;
    const double chunk = beam_partial_size(S, C, m) / (double)m;
    s.C = m;
    const uint32_t nc = live * F, kept = nc < l.width ? nc : l.width;
    for (uint32_t x = lane; x < nc; x += kBlock) { k.lb[x] = 0u; k.tb[x] = ~0u; }
    if (chunk != made_for) {   // (the m-th part of m chunks is nearly always the same)
      setup = shared_table<true>(s, chunk, scf, tab);
      made_for = chunk;
    }
    __syncthreads();
    if (!setup.ok) {
      if (lane == 0u) {   // from the start, as beam_init_kernel leaves it
        *live_p = 1u;
        (ws + l.off_rank[0])[i * l.width] = 0u;
        atomicMax(&g_marked_call, call);
      }
      return;
    }
    const double longest = (double)m * setup.t_max * (1.0 + 1e-9);
    const bool prune = nc > kBlock && longest + 0.25 * setup.t_min > longest && longest < inf64() &&
                       setup.t_min > 1e-30;
    if (prune) {
      // 64 / live lanes (a power of two) add up a kept schedule's chunks
      const uint32_t shift = (uint32_t)__clz((int)(live - 1u)) - 26u, part = lane & ((1u << shift) - 1u);
      const uint32_t p = lane >> shift;
      SharedBound sum;
      if (p < live)
        for (uint32_t c = part; c + 1u < m; c += 1u << shift) sum.add(tab, k.orders[half][p][c] & 31u, both);
      for (int off = 1; off < (1 << shift); off <<= 1) sum.join(off, both);
      if (p < live && part == 0u) k.prefix(p) = sum;
      __syncthreads();
      for (uint32_t x = lane; x < nc; x += kBlock) {
        const uint32_t p = by_orders(x);
        SharedBound lb = k.prefix(p);
        lb.add(tab, tab.rank_of[x - p * F], both);
        k.lb[x] = __float_as_uint(fmaxf(lb.value(both), 0.0f));
      }
    }
    __syncthreads();
    // at most 64 with the lowest bounds (none of them, if more are equal: then any)
    uint32_t most = 0xfffffffeu;
    if (prune) {
      const uint32_t beyond = beam_kth<kMost>(k.lb, nc, kBlock + 1u);
      uint64_t below = 0ull;
      for (uint32_t x = lane; x < nc; x += kBlock) below |= k.lb[x] < beyond ? 1ull : 0ull;
      most = __builtin_amdgcn_ballot_w64(below != 0ull) != 0ull ? beyond - 1u : most;
    }
    bool bad = false;
    for (uint32_t round = 0; round <= nc; ++round) {
      const uint32_t got = beam_gather(k.lb, nc, most, kBlock, k.list);
      if (got == 0u) break;
      __syncthreads();
      if (lane < got) {
        const uint32_t x = k.list[lane], p = by_orders(x);
        const uint32_t last = tab.rank_of[x - p * F];
        const uint32_t* row = (const uint32_t*)k.orders[half][p];
        LaneLds lds;
        lds.base = block + LayoutRing::lane_term_rec(lane);
        lds.aux = block + kCap * 128u + (LayoutRing::lane_term_tail(lane) - LayoutRing::kRecBytes);
        uint32_t four = 0u;
        auto rank_at = [&](uint32_t c) {
          four = (c & 3u) == 0u ? row[c >> 2] : four >> 8;
          return c + 1u == m ? last : four & 0xffu;
        };
        const SharedModel model(tab, setup, s.ctype, rank_at);
        const FastResult r = shared_ring<true>(s, model, lds);
        bad = bad || !r.ok;
        k.time[x] = r.t_done;
        // (a NaN or negative time is not possible where r.ok)
        k.tb[x] = __float_as_uint((float)r.t_done * (1.0f + 1e-6f));
        k.lb[x] = ~0u;
      }
      __syncthreads();
      if (prune) {
        const uint32_t limit = beam_kth<kMost>(k.tb, nc, kept);
        most = limit < 0xfffffffeu ? limit : 0xfffffffeu;
      }
    }
    // a simulation that gave up: the scenario has no answer
    if (__builtin_amdgcn_ballot_w64(bad) != 0ull) { live = 0u; break; }
    // the candidates that may be among the kept ones, then each one's place
    const uint32_t last = beam_kth<kMost>(k.tb, nc, kept);
    const uint32_t left = beam_gather(k.tb, nc, last, nc, k.list);
    __syncthreads();
    for (uint32_t a = lane; a < left; a += kBlock) {
      const uint32_t x = k.list[a], px = by_orders(x), jx = x - px * F;
      const uint32_t kx = jx * kBeamMaxWidth + k.rank[px];
      const double tx = k.time[x];
      uint32_t before = 0u;
      for (uint32_t o = 0; o < left; ++o) {
        const uint32_t y = k.list[o], py = by_orders(y), jy = y - py * F;
        const double ty = k.time[y];
        before += (ty < tx || (ty == tx && jy * kBeamMaxWidth + k.rank[py] < kx)) ? 1u : 0u;
      }
      if (before < kept) {
        k.key[before] = (uint16_t)kx;
        k.parent[before] = (uint8_t)px;
        if (before == 0u) ((double*)(ws + l.off_best))[i] = tx;
      }
    }
    __syncthreads();
    if (lane < kept) {
      uint32_t smaller = 0u;
      for (uint32_t q = 0; q < kept; ++q) smaller += k.key[q] < k.key[lane] ? 1u : 0u;
      k.rank[lane] = (uint8_t)smaller;
    }
    for (uint32_t q = 0; q < kept; ++q)
      if (lane < m)   // (a lane per chunk: at most 64)
        k.orders[half ^ 1u][q][lane] =
            lane + 1u < m ? k.orders[half][k.parent[q]][lane] : tab.rank_of[k.key[q] / kBeamMaxWidth];
    live = kept;
    __syncthreads();
  }
  if (live != 0u && lane < C) {
    const uint32_t rank = k.orders[(C & 1u) ^ 1u][0][lane];
    uint32_t digit = 0u;   // the permutation's number among those of D dimensions
    for (uint32_t j = 1; j < F; ++j) digit = tab.rank_of[j] == rank ? j : digit;
    (ws + l.off_digits[C & 1u])[i * l.width * l.mc + lane] = (uint8_t)digit;
  }
  if (lane == 0u) *live_p = live != 0u ? kBeamDone : 0u;
}

// The better of the beam's best schedule and the greedy plan (the beam's on
// equal times); NaN / all-ones for scenarios without an answer.
__global__ void __launch_bounds__(256)
beam_finish_kernel(themis_batch_t b, BeamLayout l, const uint8_t* __restrict__ ws,
                   double* __restrict__ best_t, uint8_t* __restrict__ best_orders) {
  const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= b.n) return;
  const uint32_t live = ((const uint32_t*)(ws + l.off_live))[i];
  const uint32_t D = b.ndims[i], C = b.chunks[i];
  const double tb = ((const double*)(ws + l.off_best))[i];
  const double tg = ((const double*)(ws + l.off_greedy_t))[i];
  const bool ok = live != 0u && tg == tg;
  const bool greedy = ok && tg < tb;
  best_t[i] = ok ? (greedy ? tg : tb) : nan64();
  if (!best_orders) return;
  // step m reads buffer (m - 1) & 1 and writes the other: a scenario's last step is m = C
  const uint8_t* digits = ws + l.off_digits[C & 1u] + i * l.width * l.mc;
  const uint8_t* plan = ws + l.off_greedy_orders + i * l.mc;
  for (uint32_t c = 0; c < b.max_chunks; ++c) {
    uint32_t code = 0xFFu;
    if (ok && c < C) code = greedy ? plan[c] : nth_permutation_code(D, digits[c]);
    best_orders[i * b.max_chunks + c] = (uint8_t)code;
  }
}

// ---------------------------------------------------------------------------
// themis_metrics_batch: average bandwidth utilisation (Sec. 3) and Ideal
// (Table 3) per scenario.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
metrics_kernel(themis_batch_t b, const double* __restrict__ t_done,
               const double* __restrict__ transfer, double* __restrict__ utilization,
               double* __restrict__ ideal) {
  uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= b.n) return;
  const int D = b.ndims[i];
  double u = nan64(), id = nan64();
  if (D >= 1 && D <= kMaxDims) {
    double num = 0.0, den = 0.0;
    for (int k = 0; k < D; ++k) {
      const double bw = b.bw[(size_t)k * b.n + i];
      num = num + transfer[(size_t)k * b.n + i] * bw;
      den = den + bw;
    }
    double total = 0.0;
    if (b.n_coll) {
      const uint32_t Q = b.n_coll[i] <= b.max_coll ? b.n_coll[i] : b.max_coll;
      for (uint32_t q = 0; q < Q; ++q) total = total + b.coll_size[(size_t)q * b.n + i];
    } else {
      total = b.size_bytes[i];
    }
    u = num / (t_done[i] * den);
    id = total / den;
  }
  if (utilization) utilization[i] = u;
  if (ideal) ideal[i] = id;
}

// ---------------------------------------------------------------------------
// themis_classify_batch: bandwidth provisioning class of each dimension pair
// (Sec. 6.3).  classes [6][n].
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
classify_kernel(themis_batch_t b, uint8_t* __restrict__ classes) {
  const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= b.n) return;
  const int D = b.ndims[i];
  bool ok = D >= 1 && D <= kMaxDims;
  double P[kMaxDims], B[kMaxDims];
#pragma unroll
  for (int k = 0; k < kMaxDims; ++k) {
    const uint32_t p = b.npus[(size_t)k * b.n + i];
    P[k] = (double)p;
    B[k] = b.bw[(size_t)k * b.n + i];
    if (k < D && !(p >= 2u && finite_positive(B[k]))) ok = false;
  }
  int pair = 0;
#pragma unroll
  for (int K = 0; K < kMaxDims; ++K) {
    double shrink = 1.0;  // factor by which a chunk shrinks between dimK and dimL
#pragma unroll
    for (int L = K + 1; L < kMaxDims; ++L, ++pair) {
      shrink = shrink * P[L - 1];
      const double balanced = shrink * B[L];
      uint32_t c = B[K] < balanced ? THEMIS_BW_OVER_PROVISIONED
                 : B[K] > balanced ? THEMIS_BW_UNDER_PROVISIONED
                                   : THEMIS_BW_JUST_ENOUGH;
      if (!ok || L >= D) c = 0xFFu;
      classes[(size_t)pair * b.n + i] = (uint8_t)c;
    }
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
constexpr uint32_t kMaxSlots = 32767u;  // 16-bit queue entries, all-ones reserved

static int check_batch(const themis_batch_t* b, bool need_intra, bool need_inter) {
  if (!b) return THEMIS_ERR_INVALID_ARGUMENT;
  if (b->max_chunks < 1u || b->max_chunks > THEMIS_MAX_CHUNKS) return THEMIS_ERR_INVALID_ARGUMENT;
  if (b->threshold_mode != THEMIS_THR_ABS && b->threshold_mode != THEMIS_THR_REL)
    return THEMIS_ERR_INVALID_ARGUMENT;
  if (b->n == 0) return THEMIS_OK;
  if (!b->ndims || !b->npus || !b->bw || !b->chunks) return THEMIS_ERR_INVALID_ARGUMENT;
  if (need_inter && (!b->inter_policy || !b->threshold)) return THEMIS_ERR_INVALID_ARGUMENT;
  if (need_intra && !b->intra_policy) return THEMIS_ERR_INVALID_ARGUMENT;
  if (b->n_coll) {
    if (!b->coll_size || b->max_coll < 1u) return THEMIS_ERR_INVALID_ARGUMENT;
    if ((uint64_t)b->max_coll * b->max_chunks > kMaxSlots) return THEMIS_ERR_UNSUPPORTED;
  } else if (!b->size_bytes) {
    return THEMIS_ERR_INVALID_ARGUMENT;
  }
  if (b->n > (uint64_t)0x7fffffff * kBlock) return THEMIS_ERR_UNSUPPORTED;
  return THEMIS_OK;
}

// Compute units of the current device (0 if the query fails: callers then take
// the variant that suits large grids).
static unsigned compute_units() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  return cus > 0 ? (unsigned)cus : 0u;
}

// Number of a call whose kernels may hand evaluations over (see g_marked_call).
static unsigned long long next_call_number() {
  static std::atomic<unsigned long long> counter{0};
  return ++counter;
}

// Launches through hipLaunchKernel and keeps the first error that a launch of
// this call returns: the process-wide "last error" may hold what an unrelated
// earlier call of the host program left there, and reading it would take that
// away from its owner.
struct Launcher {
  hipStream_t stream;
  hipError_t first = hipSuccess;
  explicit Launcher(void* s) : stream((hipStream_t)s) {}
  template <typename... P, typename... A>
  void operator()(void (*kernel)(P...), unsigned blocks, unsigned threads, A&&... a) {
    with_lds(0u, kernel, blocks, threads, std::forward<A>(a)...);
  }
  // Dynamic LDS, and as many workgroups as there are: the kernel numbers them with block_index().
  template <typename... P, typename... A>
  void in_rows(unsigned lds_bytes, void (*kernel)(P...), uint64_t blocks, unsigned threads, A&&... a) {
    const uint64_t rows = (blocks + kGridRow - 1u) / kGridRow;
    if (rows > (1ull << 32) / kGridRow) {   // (block_index() has 32 bits)
      if (first == hipSuccess) first = hipErrorInvalidConfiguration;
      return;
    }
    launch(lds_bytes, kernel, rows > 1u ? dim3(kGridRow, (unsigned)rows) : dim3((unsigned)blocks), threads,
           std::forward<A>(a)...);
  }
  template <typename... P, typename... A>
  void with_lds(unsigned lds_bytes, void (*kernel)(P...), unsigned blocks, unsigned threads, A&&... a) {
    launch(lds_bytes, kernel, dim3(blocks), threads, std::forward<A>(a)...);
  }
  int status() const { return first == hipSuccess ? THEMIS_OK : THEMIS_ERR_DEVICE; }

 private:
  template <typename... P, typename... A>
  void launch(unsigned lds_bytes, void (*kernel)(P...), dim3 grid, unsigned threads, A&&... a) {
    std::tuple<P...> params(std::forward<A>(a)...);  // converted to the kernel's own parameter types
    void* ptrs[sizeof...(P)];
    fill(ptrs, params, std::index_sequence_for<P...>{});
    const hipError_t e = hipLaunchKernel((const void*)kernel, grid, dim3(threads), ptrs, lds_bytes, stream);
    if (first == hipSuccess) first = e;
  }
  template <typename T, size_t... I>
  static void fill(void** ptrs, T& params, std::index_sequence<I...>) {
    ((ptrs[I] = (void*)&std::get<I>(params)), ...);
  }
};

using SimKernel = void (*)(themis_batch_t, const uint8_t*, double*, void*, int, double*,
                           unsigned long long);

template <typename L, int kMode>
static SimKernel pick_flags(bool busy, bool fix) {
  return busy ? (fix ? simulate_kernel<L, kMode, true, true> : simulate_kernel<L, kMode, true, false>)
              : (fix ? simulate_kernel<L, kMode, false, true> : simulate_kernel<L, kMode, false, false>);
}

// Queue-entry store modes of the lanes' loops (8-bit entries: up to 64 chunks).
template <typename L>
static SimKernel pick_mode(int mode, bool busy, bool fix) {
  return mode == kNoQueueOrder ? pick_flags<L, kNoQueueOrder>(busy, fix)
       : mode == kBytes ? pick_flags<L, kBytes>(busy, fix) : pick_flags<L, kWords>(busy, fix);
}

// Smallest LDS layout that holds max_chunks chunks per evaluation (the less
// LDS a wavefront takes, the more of them share a CU).
static uint32_t layout_capacity(uint32_t max_chunks) {
  return max_chunks > 256u ? 512u : max_chunks > 128u ? 256u : max_chunks > 64u ? 128u
       : max_chunks > 16u ? 64u : 16u;
}

static SimKernel pick_simulate_kernel(uint32_t cap, int mode, bool busy, bool fix, bool two) {
  return cap == 16u ? (two ? pick_mode<TwoPerSimd<Layout16>>(mode, busy, fix) : pick_mode<Layout16>(mode, busy, fix))
                    : (two ? pick_mode<TwoPerSimd<LayoutRing>>(mode, busy, fix) : pick_mode<LayoutRing>(mode, busy, fix));
}

// The same with four lanes per scenario.
template <uint32_t kChunks>
static SimKernel pick_quad_mode(int mode, bool fix) {
  using L = LayoutQuad<kChunks, 16>;
  constexpr int kOne = kChunks <= 128u ? kBytes : kShorts, kTwo = kChunks >= 128u ? kShorts : kBytes;
  constexpr bool kOthers = kChunks <= 64u;
#define THEMIS_QUAD_KERNEL(MODE) \
  (fix ? simulate_quad_kernel<L, MODE, true, kOthers> : simulate_quad_kernel<L, MODE, false, kOthers>)
  return mode == kNoQueueOrder ? THEMIS_QUAD_KERNEL(kNoQueueOrder) : mode == kShorts ? THEMIS_QUAD_KERNEL(kTwo)
                                                                                     : THEMIS_QUAD_KERNEL(kOne);
#undef THEMIS_QUAD_KERNEL
}
static SimKernel pick_quad_kernel(uint32_t cap, int mode, bool fix) {
  return cap <= 64u ? pick_quad_mode<64>(mode, fix) : cap == 128u ? pick_quad_mode<128>(mode, fix)
       : cap == 256u ? pick_quad_mode<256>(mode, fix) : pick_quad_mode<512>(mode, fix);
}

// Into how many shares the follow-up kernel divides a window's turns.  A share of many turns is
// one after the other, and every share looks at the whole window: eight for every workgroup
// that the GPU holds and at most one for each turn (any NPU counts, two / eight, us: 100,003 4-D
// ragged scenarios of 64 chunks 1,164 / 855, 100,003 of 24 824 / 734, 1,048,576 with 10,000 of
// other counts 2,614 / 2,640); where turns are short, of two turns unless there are too few
// windows.
static uint32_t follow_up_shares(uint64_t n, uint32_t max_chunks) {
  const uint64_t resident = 4u * (compute_units() ? compute_units() : 256u), windows = (n + kWindow - 1u) / kWindow;
  auto shares_for = [&](uint64_t items) { return std::min<uint64_t>(kWindowTurns, (items + windows - 1u) / windows); };
  const uint64_t shares = shares_for(8u * resident);
  return (uint32_t)(max_chunks > 8u ? shares : std::min(shares, std::max<uint64_t>(kWindowTurns / 2u, shares_for(2u * resident))));
}

// The generic area comes first in the workspace, rounded up so that the trace
// regions behind it keep the workspace's alignment up to 64 bytes.
static size_t generic_area_bytes(uint64_t evals, uint64_t slots) {
  return (workspace_bytes(evals, slots) + 63u) & ~(size_t)63u;
}

static unsigned blocks_for(uint64_t items) { return (unsigned)((items + kBlock - 1) / kBlock); }

// Grid of a follow-up kernel (its workgroups stride over the groups of 64
// evaluations): enough to fill the device, no more.
static unsigned follow_up_blocks(uint64_t items) {
  const unsigned cus = compute_units();
  const uint64_t cap = 8u * (cus ? cus : 256u), all = (items + kBlock - 1u) / kBlock;
  return (unsigned)(all < cap ? all : cap);
}

// Which mapping themis_sweep's LDS kernel uses for a layout capacity: beyond 64
// chunks four lanes per evaluation, where LDS held back the lanes (four wavefronts
// per CU at 128 chunks, three at 256, two at 512; quads 16, 12 and 8).  Measured (us, a
// lane each, as long as there was that / quads): 100 chunks, all schedulers and 8 thresholds,
// 300 4-D scenarios 506 / 246, 30,000 2,208 / 1,389; 60,000 of 128 chunks, Themis schedulers,
// 5,400 / 3,490; 70 chunks 2,734 / 1,555; 30,001 of 200 chunks 10,508 / 3,890.  Up to 64 chunks
// the lanes, twelve wavefronts per CU, are faster where they fill the GPU (64 chunks, all
// schedulers, 30,000 4-D scenarios 712 / 858, on one network 697 / 969), and slower where
// they do not (2,000 366 / 212, 244 of 52 chunks 279 / 132).
static std::atomic<int> sweep_mapping{THEMIS_MAPPING_AUTO};
static bool sweep_mapping_is_quad(uint32_t cap) {
  const int forced = sweep_mapping.load(std::memory_order_relaxed);
  return cap > 64u || forced == THEMIS_MAPPING_QUAD;
}

// Four lanes per scenario (themis_quad.hpp) or one?  A pass of the quads' loop
// takes a wavefront some 860 clocks on its own and a SIMD 350, for 16 scenarios;
// the lanes' loop takes 1,300 and 620 for 64.  So quads are faster until the
// lanes fill the GPU (a wavefront on each SIMD: 65,536 scenarios on 256 CUs), and beyond 64
// chunks always, where LDS held back the lanes (a lane each, before there were only
// quads: 250 chunks 20,001 scenarios 1,530 us, 712 on quads).  Measured (us, simulation
// with queue orders, quads / lanes), 64 chunks:
//   4-D Smallest-Chunk-First    32,768 184 / 334, 65,536 271 / 346, 70,000 358 / 397, 131,072 498 / 411
//   the same on one network     32,768 184 / 299, 65,536 281 / 310, 70,000 365 / 345, 131,072 510 / 362
//   3-D first-in-first-out      32,768 128 / 272, 65,536 177 / 280, 70,000 242 / 324, 131,072 327 / 343
//   3-D, other NPU counts       32,768 157 / 572, 65,536 224 / 589, 70,000 300 / 631, 131,072 412 / 629
// and 8 chunks, 4-D Smallest-Chunk-First: 32,768 32 / 62, 65,536 46 / 62, 131,072 79 / 72.  Other
// counts on four dimensions are left to the follow-up kernel either way (65,536 972 / 945).
// Above the line lanes are up to 1.4 times as fast on a network that all scenarios share, and
// quads up to 2.1 times on other NPU counts, which the host does not see.
static bool simulate_on_quads(uint64_t n, uint32_t cap) {
  const int forced = sweep_mapping.load(std::memory_order_relaxed);
  const uint64_t lanes = 4u * (uint64_t)kBlock * (compute_units() ? compute_units() : 256u);
  return cap > 64u || (forced != THEMIS_MAPPING_AUTO ? forced == THEMIS_MAPPING_QUAD : n <= lanes);
}

// Whole wavefronts per scenario (themis_wave.hpp) or not?  A wavefront's event costs a
// SIMD some 300 clocks (three resident wavefronts), one alone takes 560.  What runs above
// the line is quads: 860 clocks a pass for 16 scenarios, whatever their number until
// every SIMD has a wavefront of them.  Simulation with queue orders (us, wavefront / quads), four
// dimensions, Smallest-Chunk-First, powers of two:
//   8 chunks     512 24 / 29, 2,048 28 / 26, 3,072 32 / 26, 4,096 37 / 27, 8,192 61 / 28
//   64 chunks    512 121 / 183, 2,048 142 / 158, 3,072 166 / 158, 4,096 195 / 158, 8,192 341 / 168
//   250 chunks   512 460 / 693, 2,048 547 / 593, 3,072 1,000 / 593, 4,096 1,142 / 595
// Other NPU counts: 8 chunks 4,096 38 / 58, 64 chunks 4,096 196 / 209, 8,192 343 / 224, 250 chunks
// 2,048 547 / 677, 4,096 1,140 / 678.  So the line is where other counts of up to 64 chunks are
// the same on both sides (the host does not see the counts); powers of two are up to 1.4 times as fast
// on quads from 2,500 scenarios on, and beyond 64 chunks, where LDS holds eight wavefronts
// a CU, both are up to 1.9 times from 2,049 on.
// Planner (us, wavefront / lane): 2,048 23 / 26, 4,096 36 / 26 (other counts 24 / 144, 36 / 149);
// 3,072 28 / 26 on four dimensions (28 / 147), 19 / 26 on two, 11 / 26 on one.
constexpr uint64_t kWaveSimulate = 4096, kWavePlan = 3072;
constexpr uint64_t kMostWavefronts = 0xffffffffull / kBlock;   // of a launch with a workgroup each
static std::atomic<int> batch_mapping{THEMIS_MAPPING_AUTO};
static bool on_wavefronts(uint64_t items, uint64_t most) {
  const int forced = batch_mapping.load(std::memory_order_relaxed);
  return forced != THEMIS_MAPPING_AUTO ? forced == THEMIS_MAPPING_WAVE && items <= kMostWavefronts
                                       : items <= most;
}
// Wavefronts of plan_kernel for 64 scenarios: four where one each would leave the
// SIMDs with two or fewer (64 chunks, us, one / four: 65,536 4-D scenarios of other
// NPU counts 177 / 89, 100,003 of them 205 / 126, ragged ones 163 / 100; 65,536 of powers
// of two 38 / 40, 100,003 42 / 45).
static unsigned plan_waves(uint64_t n) {
  return blocks_for(n) <= 8u * (compute_units() ? compute_units() : 256u) ? kPlanWaves : 1u;
}
static bool plan_on_wavefronts(uint64_t items) { return on_wavefronts(items, kWavePlan); }
static bool simulate_on_wavefronts(uint64_t items) { return on_wavefronts(items, kWaveSimulate); }

// LDS of the launches that simulate a batch of traces with a wavefront each (0:
// none).  How much a trace needs depends on its dimensions and NPU counts, which
// the host does not see: the first launch has enough for up to three dimensions
// of powers of two, the second also for four, and for three of other counts, the
// third for what fits at all; each takes what the one before has left marked.
// One launch does where all the traces are resident with the larger blocks.
struct TraceWaveLaunches {
  uint32_t lds[3];
};
constexpr uint32_t kLdsOfCu = 160u * 1024u;
// (four wavefronts on a SIMD by their registers)
static uint64_t trace_wave_resident(uint32_t lds) {
  const uint64_t per_cu = lds ? kLdsOfCu / lds : 0u;
  return (per_cu < 16u ? per_cu : 16u) * (compute_units() ? compute_units() : 256u);
}
static TraceWaveLaunches trace_wave_launches(uint64_t n, uint32_t slots, uint32_t max_coll) {
  const uint32_t most4 = kTraceMaxRanks / (trace_wave_row(4u, true) / 4u);
  TraceWaveLaunches t;
  t.lds[0] = trace_wave_layout(slots, 3u, max_coll, true, false).bytes;
  t.lds[1] = std::max(trace_wave_layout(slots, 3u, max_coll, true, true).bytes,
                      trace_wave_layout(slots, 4u, max_coll, true, false).bytes);
  t.lds[2] = std::max(t.lds[1], trace_wave_layout(slots, 4u, std::min(max_coll, most4), true, true).bytes);
  for (int j = 1; j < 3; ++j)
    if (t.lds[j] > kLdsOfCu || t.lds[j] == t.lds[j - 1]) t.lds[j] = t.lds[j] > kLdsOfCu ? kLdsOfCu : 0u;
  if (t.lds[0] > kLdsOfCu) t.lds[0] = 0u;
  for (int j = 2; j > 0; --j)
    if (t.lds[j] != 0u && n <= trace_wave_resident(t.lds[j]))
      for (int i = 0; i < j; ++i) t.lds[i] = 0u;
  return t;
}
// How a batch of traces is simulated.  On wavefronts an event of a trace takes 0.42
// us and 18 ns more per wavefront of its CU; they take turns where the LDS of a CU
// holds fewer than there are traces.  On quads it takes 0.65 us, up to 0.9 where
// they fill the GPU (16,384 traces).  With a lane each it takes 1.5 us and up, 5.2
// with release times, up to a wavefront of them per CU.  Measured (ms, wavefront /
// quad / lane; three dimensions unless said):
//   200 collectives of 64 chunks   64 traces 31 / 50 / 110, 1,024 68 / 52 / 117, 16,384 - / 68 / 139
//   100 of 32                      1,024 11.0 / 13.2 / 28.5, 4,096 29 / 13 / 30, 16,384 97 / 17.5 / 35
//   50 of 32                       1,500 6.4 / 6.4 / 14.4, 3,000 7.1 / 6.4 / 14.5, 65,536 - / 22 / 87
//   50 of 32, releases             64 4.1 / - / 49, 2,048 6.1 / - / 54, 16,384 28 / - / 55
//   40 of 16, four dimensions      2,048 4.2 / 4.1 / 8.8, 16,384 21 / 5.9 / 10.9
//   4 of 8                         64 0.11 / 0.16 / 0.33, 4,096 0.17 / 0.16 / 0.35
// Quads take what is released together on powers of two; what they leave (the
// host does not see the NPU counts) goes to wavefronts or lanes as if they were not.
struct TracePlan {
  bool waves, quads, waves_after;
};
static TracePlan trace_plan(const themis_batch_t& b, uint32_t slots, uint32_t region_bytes) {
  const int batch = batch_mapping.load(std::memory_order_relaxed), lanes = sweep_mapping.load(std::memory_order_relaxed);
  const bool releases = b.release_time != nullptr;
  TracePlan p;
  p.quads = lanes != THEMIS_MAPPING_LANE && !releases && trace_quad_layout(slots, 4u, b.max_coll).region <= region_bytes &&
            trace_quad_layout(slots, 3u, b.max_coll).lds <= kLdsOfCu;
  const uint32_t lds = trace_wave_layout(slots, 3u, b.max_coll, true, false).bytes;
  if (lds > kLdsOfCu || b.n > kMostWavefronts || batch == THEMIS_MAPPING_LANE) {
    p.waves = p.waves_after = false;
    return p;
  }
  const double cus = compute_units() ? compute_units() : 256u;
  const double resident = (double)trace_wave_resident(lds) / cus;   // wavefronts of a CU
  const double per_cu = std::min(resident, std::max(1.0, (double)b.n / cus));
  const double event = std::max(1.0, (double)b.n / (cus * resident)) * (0.42 + 0.018 * per_cu);
  p.waves_after = event < (releases ? 5.2 : 1.5);
  p.waves = batch == THEMIS_MAPPING_WAVE || (p.quads ? event < 0.55 : p.waves_after);
  return p;
}

// A wavefront per evaluation in a sweep of few: what comes after it takes other NPU counts
// a lane each.  The line lies where themis_simulate_batch's does; 4,080 evaluations on four
// dimensions, us, wavefront / other mapping (powers of two on lanes, beyond 64 chunks on quads):
//   1 chunk 18 / 12 (other counts 18 / 21), 4 27 / 31 (28 / 74), 64 217 / 296 (219 / 1,790),
//   256 1,279 / 622 (1,278 / 3,547), 512 2,550 / 1,235 (2,552 / 6,500; two dimensions 1,221 / 631,
//   1,230 / 3,238).
static bool sweep_on_wavefronts(uint64_t evaluations) {
  return sweep_mapping.load(std::memory_order_relaxed) == THEMIS_MAPPING_AUTO && evaluations <= kWaveSimulate;
}

// A wavefront per scenario for the beam search (beam_kernel), or a lane per
// candidate, step by step?  A wavefront works its candidates off 64 at a time,
// up to width 4 in one round as a rule (bounds); eight of them fit a CU up to
// width 4, six up to 16.
//   - Few scenarios are faster with all candidates at once: up to two turns of
//     the per-order tables (two wavefronts per CU), which may have scenarios left
//     to them after it (40 4-D scenarios of other NPU counts, width 4, 24 chunks:
//     9.0 against 11.5 ms), and for a wider beam, which takes several rounds, up
//     to what the GPU holds (20 4-D scenarios, width 16, 48 chunks: 27 against
//     38 ms; 800, 64 chunks: 55 either way).
//   - Narrow beams leave lanes idle (24 candidates at width 1 on four dimensions,
//     6 on three), where a lane per candidate packs them: width 1 is 1.1 to 2.3
//     times slower by scenario on three and four dimensions of power-of-two NPU
//     counts (24 chunks, 4,096 scenarios: 4.2 against 2.8 ms), widths 2 and 3 are
//     0.65 to 0.98 of it in one turn and up to 1.3 beyond it on four dimensions.
//   - Width 4 on four dimensions, 24 chunks: 700 to 900 scenarios 1.06 to 1.10,
//     1,100 to 2,048 0.87 to 1.02, 2,100 to 2,700 (a second turn, nearly empty)
//     1.06 to 1.09, 4,096 0.94; widths 5 to 8 0.80 in a full turn, up to 1.14 off
//     one; width 12 0.66 to 0.90.  On two and three dimensions all of these are
//     0.2 to 0.7, and on other NPU counts of up to three 0.1 to 0.3, so they stay.
static bool beam_by_scenario(uint64_t n, uint64_t lane_waves, uint32_t width) {
  const uint64_t cus = compute_units() ? compute_units() : 256u;
  if (width == 1u) return false;
  if (width > 4u) return lane_waves > 4u * (uint64_t)LayoutRing::kWavesPerSimd * cus;
  return lane_waves > 4u * cus && (width == 4u ? n >= 4u * cus : n <= 8u * cus);
}

// Lanes per scenario in sweep_plans_kernel.
static uint32_t sweep_plans_width(int n_thr) {
  uint32_t width = 1u;
  while (width < (uint32_t)n_thr) width *= 2u;
  return width;
}

// Does themis_sweep look for thresholds that share a plan?  From four
// thresholds on, and where the sweep is more than one turn of the wavefronts
// that are resident at once: a smaller one takes the time of one wavefront
// either way.  And where there is enough to simulate for the launches it takes
// (2-D, eight thresholds: 16,384 scenarios of one chunk 27 against 25 us without,
// of two 30 against 35; 65,536 of one 47 against 60).
static bool sweep_shares_plans(uint64_t n, uint32_t max_chunks, int n_thr, unsigned policy_mask) {
  if (n_thr < 4 || n_thr > (int)kSweepJobsMaxThr || (policy_mask & ~THEMIS_SWEEP_BASELINE) == 0u) return false;
  // sweep_plans_kernel has sweep_plans_width() lanes per scenario, of a grid of less
  // than 2^32; so the number of jobs and the scenario's index fit 32 bits
  if (n > 0xfffff000ull / sweep_plans_width(n_thr)) return false;
  if (n * max_chunks < 32768u) return false;
  const uint32_t cap = layout_capacity(max_chunks);
  const bool quad = sweep_mapping_is_quad(cap);
  const uint64_t per_cu = quad ? 8u : 12u;
  const uint64_t group = quad ? kBlock / 4u : kBlock;
  const uint64_t waves = (n + group - 1u) / group *
      sweep_roles((uint32_t)n_thr, (uint32_t)__builtin_popcount(policy_mask & 7u), policy_mask);
  const unsigned cus = compute_units();
  return waves > per_cu * (cus ? cus : 256u) * 5u / 4u;
}

}  // namespace themis

using namespace themis;

extern "C" {

int themis_version(void) { return 103; }

const char* themis_status_string(int status) {
  switch (status) {
    case THEMIS_OK: return "success";
    case THEMIS_ERR_INVALID_ARGUMENT: return "invalid argument";
    case THEMIS_ERR_UNSUPPORTED: return "unsupported request";
    case THEMIS_ERR_DEVICE: return "HIP device error";
    case THEMIS_ERR_WORKSPACE: return "workspace missing, too small or misaligned, or the request exceeds the built-in scratch";
    default: return "unknown status";
  }
}

int themis_queue_entry_bytes(uint32_t max_chunks, uint32_t max_coll) {
  uint64_t slots = (uint64_t)max_chunks * (max_coll ? max_coll : 1u);
  return slots <= 127u ? 1 : 2;
}

size_t themis_workspace_bytes(uint64_t n, uint32_t max_chunks, uint32_t max_coll) {
  size_t generic = generic_area_bytes(n, (uint64_t)max_chunks * (max_coll ? max_coll : 1u));
  size_t trace = max_coll ? (size_t)n * trace_layout(max_chunks, max_coll).bytes : 0;
  return generic + trace;
}

int themis_plan_batch(const themis_batch_t* batch, uint8_t* orders, double* loads, void* stream) {
  int st = check_batch(batch, false, true);
  if (st != THEMIS_OK) return st;
  if (batch->n == 0) return THEMIS_OK;
  if (!orders) return THEMIS_ERR_INVALID_ARGUMENT;
  const TraceView tv = trace_view(*batch);
  if (batch->n * (uint64_t)tv.mc > (uint64_t)0x7fffffff * kBlock) return THEMIS_ERR_UNSUPPORTED;
  Launcher go(stream);
  if (plan_on_wavefronts(batch->n * tv.mc))
    go(plan_wave_kernel, (unsigned)(batch->n * tv.mc), kBlock, *batch, orders, loads);
  else
    go(tv.mc > 1u ? plan_kernel<true> : plan_kernel<false>,
       blocks_for(batch->n * tv.mc) * (tv.mc > 1u ? 1u : plan_waves(batch->n)), kBlock, *batch, orders, loads);
  return go.status();
}

static int simulate_batch_impl(const themis_batch_t* batch, const uint8_t* orders, double* t_done,
                               void* queue_order, double* busy, void* workspace,
                               size_t workspace_bytes_given, void* stream) {
  int st = check_batch(batch, true, false);
  if (st != THEMIS_OK) return st;
  if (batch->n == 0) return THEMIS_OK;
  if (!orders || !t_done) return THEMIS_ERR_INVALID_ARGUMENT;
  if ((uintptr_t)workspace & 15u) return THEMIS_ERR_WORKSPACE;
  const TraceView tv = trace_view(*batch);
  const bool have_ws =
      workspace != nullptr && workspace_bytes_given >= workspace_bytes(batch->n, tv.slots);
  Workspace w = carve_workspace(workspace, batch->n, tv.slots);
  const int entry_bytes =
      themis_queue_entry_bytes(batch->max_chunks, tv.on ? batch->max_coll : 0u);
  const uint32_t cap = tv.on ? 512u : layout_capacity(batch->max_chunks);
  Launcher go(stream);
  // 8-bit entries are stored four at a time by the layouts with 8-bit chunk
  // ids when the rows (2*slots bytes each) start on 4-byte boundaries
  const bool words = entry_bytes == 1 && cap <= 128u && (tv.slots & 1u) == 0u &&
                     ((uintptr_t)queue_order & 3u) == 0u;
  const int mode = !queue_order ? kNoQueueOrder
                 : entry_bytes == 2 ? kShorts : (words ? kWords : kBytes);
  if (tv.on) {
    const TraceLayout tl = trace_layout(batch->max_chunks, batch->max_coll);
    const size_t generic = generic_area_bytes(batch->n, tv.slots);
    const bool have_trace = workspace != nullptr && tl.bytes != 0u &&
                            workspace_bytes_given >= generic + (size_t)batch->n * tl.bytes;
    uint8_t* trace_area = have_trace ? (uint8_t*)workspace + generic : nullptr;
    // few wavefronts (no more than CUs): the bitmap leaves move into the LDS nothing else would use
    const bool lds_bitmaps = blocks_for(batch->n) <= compute_units();
    const bool extras = batch->release_time != nullptr || batch->fixed_delay != nullptr ||
                        queue_order != nullptr;
    auto trace_kernel = lds_bitmaps ? (extras ? simulate_trace_kernel<true, true> : simulate_trace_kernel<true, false>)
                                    : (extras ? simulate_trace_kernel<false, true> : simulate_trace_kernel<false, false>);
    unsigned long long call = 0ull;
    if (have_trace) {
      const TracePlan plan = trace_plan(*batch, tv.slots, tl.bytes);
      if (plan.waves || plan.quads) call = next_call_number();
      bool follow_up = false;
      if (!plan.waves && plan.quads)
        for (uint32_t dims : {3u, 4u}) {
          const uint32_t lds = trace_quad_layout(tv.slots, dims, batch->max_coll).lds;
          if (lds > kLdsOfCu) continue;
          go.in_rows(lds, queue_order ? simulate_trace_quad_kernel<true> : simulate_trace_quad_kernel<false>,
                     (batch->n + kBlock / 4u - 1u) / (kBlock / 4u), kBlock, *batch, orders, t_done, queue_order,
                     entry_bytes, busy, trace_area, tl.bytes, dims, follow_up, call);
          follow_up = true;
        }
      if (plan.waves || (plan.quads && plan.waves_after))
        for (uint32_t lds : trace_wave_launches(batch->n, tv.slots, batch->max_coll).lds) {
          if (lds == 0u) continue;
          go.with_lds(lds, queue_order ? simulate_trace_wave_kernel<true> : simulate_trace_wave_kernel<false>,
                      (unsigned)batch->n, kBlock, *batch, orders, t_done, queue_order, entry_bytes, busy, lds,
                      follow_up, call);
          follow_up = true;
        }
    }
    go(trace_kernel, blocks_for(batch->n), kBlock, *batch, orders, t_done, queue_order,
       entry_bytes, busy, w, have_ws, trace_area, tl, call);
    return go.status();
  }
  // Scenarios outside the LDS path (marked in t_done) go through the table
  // passes and what those leave through the generic pass: its arrays in LDS up
  // to 64 chunks, in the workspace beyond.  One launch for all of it where that
  // costs nothing: beyond 64 chunks (the generic pass needs no LDS there), with
  // a workspace (the same), and on batches small enough for every wavefront to
  // be resident whatever the LDS block (there the launches are what counts).
  // A large batch of up to 64 chunks without a workspace keeps the generic pass
  // and its 80 KiB of LDS apart from the table passes.
  const unsigned long long call = next_call_number();
  if (simulate_on_wavefronts(batch->n)) {
    // (beyond 64 chunks the generic pass asks for a workspace; without one the
    // table passes still take what they can, and the rest is NaN)
    const bool q = queue_order != nullptr, alone = batch->n <= compute_units() && (cap <= 64u || have_ws);
#define THEMIS_WAVE_KERNEL(W)                                                                        \
  (alone ? (q ? simulate_wave_kernel<W, true, true> : simulate_wave_kernel<W, false, true>)          \
         : (q ? simulate_wave_kernel<W, true, false> : simulate_wave_kernel<W, false, false>))
    go(cap <= 64u ? THEMIS_WAVE_KERNEL(1) : THEMIS_WAVE_KERNEL(8), (unsigned)batch->n, kBlock, *batch,
       orders, t_done, queue_order, entry_bytes, busy, call);
#undef THEMIS_WAVE_KERNEL
    if (alone) return go.status();
  } else if (simulate_on_quads(batch->n, cap)) {
    go.in_rows(0u, pick_quad_kernel(cap, mode, batch->fixed_delay != nullptr),
               (batch->n + kBlock / 4u - 1u) / (kBlock / 4u), kBlock, *batch, orders, t_done, queue_order,
               entry_bytes, busy, call);
  } else {
    const bool two = blocks_for(batch->n) <= 8u * (compute_units() ? compute_units() : 256u);
    go(pick_simulate_kernel(cap, mode, busy != nullptr, batch->fixed_delay != nullptr, two), blocks_for(batch->n),
       kBlock, *batch, orders, t_done, queue_order, entry_bytes, busy, call);
  }
  const Workspace ws = have_ws ? w : Workspace{};
  const uint32_t shares = follow_up_shares(batch->n, batch->max_chunks);
  const unsigned fb = follow_up_blocks(follow_up_items(batch->n, cap, shares) * kBlock);
#define THEMIS_FOLLOW_UP(MODE, CAP, G) \
  go(simulate_follow_up_kernel<MODE, CAP, G>, fb, kBlock, *batch, orders, t_done, queue_order, \
     entry_bytes, busy, ws, shares, call)
  // (8-bit entries up to 64 chunks, either up to 128, 16-bit entries beyond)
#define THEMIS_FOLLOW_UP_MODES(CAP, G)                                \
  if (mode == kNoQueueOrder) THEMIS_FOLLOW_UP(kNoQueueOrder, CAP, G); \
  else THEMIS_FOLLOW_UP(kBytes, CAP, G);
  if (cap <= 64u) {
    const bool small = blocks_for(batch->n) <= 2u * compute_units();
    if (have_ws) {
      THEMIS_FOLLOW_UP_MODES(64, 0u)
    } else if (small && cap <= 16u) {
      THEMIS_FOLLOW_UP_MODES(16, 16u)
    } else if (small) {
      THEMIS_FOLLOW_UP_MODES(64, 64u)
    } else {
      THEMIS_FOLLOW_UP_MODES(64, kNoGeneric)
      auto generic = cap <= 16u ? simulate_generic_kernel<16> : simulate_generic_kernel<64>;
      go(generic, follow_up_blocks(batch->n), kBlock, *batch, orders, t_done, queue_order, entry_bytes, busy, ws, call);
    }
  } else if (cap == 128u) {
    if (mode == kShorts) THEMIS_FOLLOW_UP(kShorts, 128, 0u);
    else THEMIS_FOLLOW_UP_MODES(128, 0u)
  } else if (cap == 256u) {
    if (mode == kNoQueueOrder) THEMIS_FOLLOW_UP(kNoQueueOrder, 256, 0u);
    else THEMIS_FOLLOW_UP(kShorts, 256, 0u);
  } else {
    if (mode == kNoQueueOrder) THEMIS_FOLLOW_UP(kNoQueueOrder, 512, 0u);
    else THEMIS_FOLLOW_UP(kShorts, 512, 0u);
  }
#undef THEMIS_FOLLOW_UP_MODES
#undef THEMIS_FOLLOW_UP
  return go.status();
}

int themis_simulate_batch(const themis_batch_t* batch, const uint8_t* orders, double* t_done,
                          void* queue_order, double* busy, void* workspace,
                          size_t workspace_bytes_given, void* stream) {
  return simulate_batch_impl(batch, orders, t_done, queue_order, busy, workspace,
                             workspace_bytes_given, stream);
}

// Device address of `scratch` on the current device, asked for once per device
// and kept: every GPU holds its own copy of the array at its own address.
static int scratch_of_current_device(void** out) {
  constexpr int kMaxDevices = 64;
  static std::atomic<void*> known[kMaxDevices];
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return THEMIS_ERR_DEVICE;
  void* p = known[dev].load(std::memory_order_acquire);
  if (!p) {
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return THEMIS_ERR_DEVICE;
    known[dev].store(p, std::memory_order_release);  // two first calls at once store the same address
  }
  *out = p;
  return THEMIS_OK;
}

int themis_simulate_batch_noalloc(const themis_batch_t* batch, const uint8_t* orders,
                                  double* t_done, void* queue_order, double* busy, void* stream) {
  int st = check_batch(batch, true, false);
  if (st != THEMIS_OK) return st;
  if (batch->n == 0) return THEMIS_OK;
  // what themis_simulate_batch would ask a caller for: traces keep their queues
  // there, single collectives only what the generic path needs beyond 64 chunks
  const bool trace = batch->n_coll != nullptr;
  const size_t need = (trace || batch->max_chunks > 64u)
      ? themis_workspace_bytes(batch->n, batch->max_chunks, trace ? batch->max_coll : 0u) : 0u;
  if (need > (size_t)THEMIS_STATIC_SCRATCH_BYTES) return THEMIS_ERR_WORKSPACE;
  void* ws = nullptr;
  st = scratch_of_current_device(&ws);
  if (st != THEMIS_OK) return st;
  // nothing in the scratch has to start at zero: the kernels initialise every
  // word they read (chunk state, list heads behind a set bitmap bit, bitmaps)
  return simulate_batch_impl(batch, orders, t_done, queue_order, busy, ws,
                             (size_t)THEMIS_STATIC_SCRATCH_BYTES, stream);
}

#define THEMIS_SWEEP_LANES(L) sweep_kernel<L,
#define THEMIS_SWEEP_QUADS(CAP) sweep_quad_kernel<CAP,
size_t themis_sweep_scratch_bytes(uint64_t n, uint32_t max_chunks, int n_thr, unsigned policy_mask) {
  if (!sweep_shares_plans(n, max_chunks, n_thr, policy_mask)) return 0;
  return kSweepJobsHeader + (size_t)n * (size_t)n_thr * sizeof(SweepJob);
}

int themis_sweep(const themis_batch_t* batch, int n_thr, const double* thr, int thr_per_scenario,
                 unsigned policy_mask, double* t_done, void* workspace,
                 size_t workspace_bytes_given, void* stream) {
  return themis_sweep_with_scratch(batch, n_thr, thr, thr_per_scenario, policy_mask, t_done, workspace,
                                   workspace_bytes_given, nullptr, 0, stream);
}

int themis_sweep_with_scratch(const themis_batch_t* batch, int n_thr, const double* thr, int thr_per_scenario,
                              unsigned policy_mask, double* t_done, void* workspace,
                              size_t workspace_bytes_given, void* scratch, size_t scratch_bytes_given,
                              void* stream) {
  int st = check_batch(batch, false, false);
  if (st != THEMIS_OK) return st;
  if (batch->n_coll) return THEMIS_ERR_UNSUPPORTED;  // sweeps are per single collective
  if (n_thr < 1 || !thr || (policy_mask & 7u) == 0u || (policy_mask & ~7u) != 0u)
    return THEMIS_ERR_INVALID_ARGUMENT;
  if (batch->n == 0) return THEMIS_OK;
  if (!t_done) return THEMIS_ERR_INVALID_ARGUMENT;
  if (((uintptr_t)workspace & 15u) || ((uintptr_t)scratch & 15u)) return THEMIS_ERR_WORKSPACE;
  int n_pol = __builtin_popcount(policy_mask & 7u);
  uint64_t evals = batch->n * (uint64_t)n_thr * (uint64_t)n_pol;
  if (evals > (uint64_t)0x7fffffff * kBlock ||
      (uint64_t)blocks_for(batch->n) * (uint64_t)(n_thr * n_pol) > 0x7fffffffull)
    return THEMIS_ERR_UNSUPPORTED;
  const bool have_ws = workspace != nullptr &&
                       workspace_bytes_given >= workspace_bytes(evals, batch->max_chunks);
  Workspace w = carve_workspace(workspace, evals, batch->max_chunks);
  const uint32_t cap = layout_capacity(batch->max_chunks);
  const bool fix = batch->fixed_delay != nullptr;
  const bool base = (policy_mask & THEMIS_SWEEP_BASELINE) != 0u;
  const bool quad = sweep_mapping_is_quad(cap);
  const uint64_t group = quad ? kBlock / 4u : kBlock;   // evaluations per wavefront
  const uint64_t groups = (batch->n + group - 1u) / group;
  if (groups * (uint64_t)(n_thr * n_pol) > 0x7fffffffull) return THEMIS_ERR_UNSUPPORTED;
  const size_t need = themis_sweep_scratch_bytes(batch->n, batch->max_chunks, n_thr, policy_mask);
  const bool share = need != 0u && scratch != nullptr && scratch_bytes_given >= need;
  const unsigned long long call = next_call_number();
  Launcher go(stream);
  SweepJobs jobs{nullptr, nullptr};
  // (one workgroup per group of scenarios and pair, the baseline once: see sweep_roles)
  const unsigned roles = sweep_roles((uint32_t)n_thr, (uint32_t)n_pol, policy_mask);
  // Layout of the quads.  The one of 256 chunks has twelve wavefronts per CU, the one
  // of 512 eight, and where these hold all of a sweep the latter is the faster by up
  // to 7 % (200 chunks, 4-D, us, 256 / 512: 600 scenarios, 646 wavefronts, 682 / 631;
  // 2,000, 2,125 wavefronts, 831 / 1,215; 30,001 4,479 / 5,595).
  const uint32_t quad_cap = !quad ? 0u : cap <= 128u ? 128u
      : groups * roles <= 8u * (compute_units() ? compute_units() : 256u) ? 512u : cap;
  auto evaluate = [&](auto kernel, uint64_t workgroups) {
    if (quad)
      go.in_rows(0u, kernel, workgroups, kBlock, *batch, n_thr, thr, thr_per_scenario, policy_mask, n_pol, t_done,
                 call, jobs);
    else
      go(kernel, (unsigned)workgroups, kBlock, *batch, n_thr, thr, thr_per_scenario, policy_mask, n_pol, t_done,
         call, jobs);
  };
  if (share) {
    uint32_t* count = (uint32_t*)scratch;
    SweepJob* list = (SweepJob*)((uint8_t*)scratch + kSweepJobsHeader);
    jobs = SweepJobs{list, count};
    const uint32_t width = sweep_plans_width(n_thr);
    go(sweep_clear_kernel, 1u, 1u, count);
    go(sweep_plans_kernel, (unsigned)((batch->n * width + kSweepPlansBlock - 1u) / kSweepPlansBlock),
       kSweepPlansBlock, *batch, n_thr, width, thr, thr_per_scenario, policy_mask, n_pol, t_done, list, count);
    // (as many workgroups as there would be jobs if all plans differed)
    const uint64_t most = (batch->n * (uint64_t)n_thr + group - 1u) / group * (uint64_t)(n_pol - (base ? 1 : 0));
#define THEMIS_SWEEP_KERNEL(K) \
  (fix ? (base ? K true, true, true> : K true, false, true>) : (base ? K false, true, true> : K false, false, true>))
    auto kernel = quad_cap == 512u ? THEMIS_SWEEP_KERNEL(THEMIS_SWEEP_QUADS(512))
                : quad_cap == 256u ? THEMIS_SWEEP_KERNEL(THEMIS_SWEEP_QUADS(256))
                : quad ? THEMIS_SWEEP_KERNEL(THEMIS_SWEEP_QUADS(128))
                : cap == 16u ? THEMIS_SWEEP_KERNEL(THEMIS_SWEEP_LANES(Layout16))
                             : THEMIS_SWEEP_KERNEL(THEMIS_SWEEP_LANES(LayoutRing));
#undef THEMIS_SWEEP_KERNEL
    evaluate(kernel, (base ? groups : 0u) + most);
  } else if (sweep_on_wavefronts(batch->n * roles)) {
    go(cap <= 64u ? sweep_wave_kernel<1> : sweep_wave_kernel<8>, (unsigned)(batch->n * roles), kBlock, *batch,
       n_thr, thr, thr_per_scenario, policy_mask, n_pol, t_done, call);
  } else {
#define THEMIS_SWEEP_KERNEL(K) \
  (fix ? (base ? K true, true, false> : K true, false, false>) : (base ? K false, true, false> : K false, false, false>))
    auto kernel = quad_cap == 512u ? THEMIS_SWEEP_KERNEL(THEMIS_SWEEP_QUADS(512))
                : quad_cap == 256u ? THEMIS_SWEEP_KERNEL(THEMIS_SWEEP_QUADS(256))
                : quad ? THEMIS_SWEEP_KERNEL(THEMIS_SWEEP_QUADS(128))
                : cap == 16u ? THEMIS_SWEEP_KERNEL(THEMIS_SWEEP_LANES(Layout16))
                             : THEMIS_SWEEP_KERNEL(THEMIS_SWEEP_LANES(LayoutRing));
#undef THEMIS_SWEEP_KERNEL
    evaluate(kernel, groups * roles);
  }
  // the follow-up passes, in one launch where themis_simulate_batch does the same
  const unsigned fb = follow_up_blocks(evals);
  const Workspace ws = have_ws ? w : Workspace{};
#define THEMIS_FOLLOW_UP(A, B, G)                                                            \
  go(share ? sweep_follow_up_kernel<A, B, G, true> : sweep_follow_up_kernel<A, B, G, false>, fb, kBlock, *batch, n_thr, thr, thr_per_scenario,      \
     policy_mask, n_pol, t_done, ws, call, jobs)
  if (cap <= 64u) {
    const bool small = blocks_for(evals) <= 2u * compute_units();
    if (have_ws) {
      THEMIS_FOLLOW_UP(0, 1, 0u);
    } else if (small && cap <= 16u) {
      THEMIS_FOLLOW_UP(0, 1, 16u);
    } else if (small) {
      THEMIS_FOLLOW_UP(0, 1, 64u);
    } else {
      THEMIS_FOLLOW_UP(0, 1, kNoGeneric);
      auto generic = cap <= 16u ? (share ? sweep_generic_kernel<16, true> : sweep_generic_kernel<16, false>)
                                : (share ? sweep_generic_kernel<64, true> : sweep_generic_kernel<64, false>);
      go(generic, fb, kBlock, *batch, n_thr, thr, thr_per_scenario, policy_mask, n_pol, t_done,
         ws, call, jobs);
    }
  } else if (cap == 128u) {
    THEMIS_FOLLOW_UP(2, -1, 0u);
  } else if (cap == 256u) {
    THEMIS_FOLLOW_UP(3, -1, 0u);
  } else {
    THEMIS_FOLLOW_UP(4, -1, 0u);
  }
#undef THEMIS_FOLLOW_UP
  if (share)
    go(sweep_spread_kernel, fb, 256, *batch, jobs, n_thr, thr, thr_per_scenario, policy_mask, n_pol, t_done, call);
  return go.status();
}

int themis_set_sweep_mapping(int mapping) {
  if (mapping != THEMIS_MAPPING_AUTO && mapping != THEMIS_MAPPING_LANE &&
      mapping != THEMIS_MAPPING_QUAD)
    return THEMIS_ERR_INVALID_ARGUMENT;
  sweep_mapping.store(mapping, std::memory_order_relaxed);
  return THEMIS_OK;
}

int themis_set_batch_mapping(int mapping) {
  if (mapping != THEMIS_MAPPING_AUTO && mapping != THEMIS_MAPPING_LANE && mapping != THEMIS_MAPPING_WAVE)
    return THEMIS_ERR_INVALID_ARGUMENT;
  batch_mapping.store(mapping, std::memory_order_relaxed);
  return THEMIS_OK;
}

size_t themis_search_workspace_bytes(uint64_t n, uint64_t max_assignments) {
  return (size_t)n * max_assignments * sizeof(double);
}

int themis_search_batch(const themis_batch_t* batch, uint64_t max_assignments, double* best_t,
                        uint8_t* best_orders, void* workspace, size_t workspace_bytes_given,
                        void* stream) {
  int st = check_batch(batch, true, false);
  if (st != THEMIS_OK) return st;
  if (batch->n_coll) return THEMIS_ERR_UNSUPPORTED;  // single collectives only
  if (max_assignments < 1u) return THEMIS_ERR_INVALID_ARGUMENT;
  if (batch->n == 0) return THEMIS_OK;
  if (!best_t) return THEMIS_ERR_INVALID_ARGUMENT;
  if (max_assignments > ((uint64_t)1 << 40) / batch->n) return THEMIS_ERR_UNSUPPORTED;
  const uint64_t evals = batch->n * max_assignments;
  if (evals > (uint64_t)0x7fffffff * kBlock || batch->n > 0x7fffffffull) return THEMIS_ERR_UNSUPPORTED;
  if (!workspace || ((uintptr_t)workspace & 7u) ||
      workspace_bytes_given < themis_search_workspace_bytes(batch->n, max_assignments))
    return THEMIS_ERR_WORKSPACE;
  double* times = (double*)workspace;
  Launcher go(stream);
  const unsigned long long call = next_call_number();
  // One wavefront per 64 assignments where the GPU holds all of them in two
  // turns (twelve wavefronts per CU): a single round, nothing to be gained from
  // bounds.  Else one per scenario, or several as long as each has some 512
  // assignments to rule out.
  const uint64_t room = 12u * (uint64_t)(compute_units() ? compute_units() : 256u);
  const uint64_t groups = (max_assignments + kBlock - 1u) / kBlock;
  uint64_t parts = groups;
  const bool tiny = max_assignments <= kSearchFew && batch->n > room;
  if (!tiny && groups > 2u * room / batch->n) {
    parts = room / batch->n;
    if (parts > max_assignments / 512u) parts = max_assignments / 512u;
    if (parts < 1u) parts = 1u;
  }
  const bool few = batch->max_chunks <= 16u, wide = max_assignments > 0x7fffffffull;
  if (tiny) {
    const bool fix = batch->fixed_delay != nullptr;
    const uint64_t per = kBlock / max_assignments, lane_blocks = (batch->n + per - 1u) / per;
    // (eight turns of wavefronts for the others: enough to even out, few to look in vain)
    uint64_t group = batch->n / (8u * room);
    group = group < 1u ? 1u : group > kBlock ? kBlock : group;
    auto search = few ? (fix ? search_few_kernel<Layout16, true> : search_few_kernel<Layout16, false>)
                      : (fix ? search_few_kernel<LayoutRing, true> : search_few_kernel<LayoutRing, false>);
    go(search, (unsigned)(lane_blocks + (batch->n + group - 1u) / group), kBlock, *batch, (uint32_t)max_assignments,
       (uint32_t)lane_blocks, (uint32_t)group, times, best_t, best_orders, call);
  } else {
    auto search = few ? (wide ? search_kernel<16, uint64_t> : search_kernel<16, uint32_t>)
                      : (wide ? search_kernel<64, uint64_t> : search_kernel<64, uint32_t>);
    go(search, (unsigned)(batch->n * parts), kBlock, *batch, max_assignments, (uint32_t)parts, times, best_t,
       best_orders, call);
  }
  go(search_table_kernel, follow_up_blocks(evals), kBlock, *batch, max_assignments, times,
     (const double*)best_t, call);
  go(search_finish_kernel, (unsigned)(batch->n < room ? batch->n : room), kBlock, *batch, max_assignments,
     (uint32_t)parts, (const double*)times, best_t, best_orders, call);
  return go.status();
}

size_t themis_beam_workspace_bytes(uint64_t n, uint32_t max_chunks, uint32_t width) {
  if (width < 1u || width > kBeamMaxWidth) return 0;
  return beam_layout(n, max_chunks, width).bytes;
}

int themis_beam_search_batch(const themis_batch_t* batch, uint32_t width, double* best_t,
                             uint8_t* best_orders, void* workspace, size_t workspace_bytes_given,
                             void* stream) {
  int st = check_batch(batch, false, true);
  if (st != THEMIS_OK) return st;
  if (batch->n_coll) return THEMIS_ERR_UNSUPPORTED;  // single collectives only
  if (width < 1u || width > kBeamMaxWidth) return THEMIS_ERR_INVALID_ARGUMENT;
  if (batch->max_chunks > 64u) return THEMIS_ERR_UNSUPPORTED;
  if (batch->n == 0) return THEMIS_OK;
  if (!best_t || !batch->intra_policy) return THEMIS_ERR_INVALID_ARGUMENT;
  const BeamLayout l = beam_layout(batch->n, batch->max_chunks, width);
  const uint64_t lanes = batch->n * (uint64_t)width * kBeamOrders;
  if (lanes > (uint64_t)0x7fffffff * kBlock || batch->n > 0x7fffffffull) return THEMIS_ERR_UNSUPPORTED;
  if (!workspace || ((uintptr_t)workspace & 63u) || workspace_bytes_given < l.bytes)
    return THEMIS_ERR_WORKSPACE;
  uint8_t* ws = (uint8_t*)workspace;
  // the greedy plan and its time (every scenario up to 64 chunks runs without a workspace)
  uint8_t* plan = ws + l.off_greedy_orders;
  double* plan_t = (double*)(ws + l.off_greedy_t);
  st = themis_plan_batch(batch, plan, nullptr, stream);
  if (st != THEMIS_OK) return st;
  st = simulate_batch_impl(batch, plan, plan_t, nullptr, nullptr, nullptr, 0, stream);
  if (st != THEMIS_OK) return st;
  const bool fix = batch->fixed_delay != nullptr;
  Launcher go(stream);
  const unsigned per_scenario = (unsigned)((batch->n + 255) / 256);
  const bool by_scenario = beam_by_scenario(batch->n, blocks_for(lanes), width);
  int half = 0;
  if (by_scenario) {
    const unsigned long long call = next_call_number();
    // (the width says how much LDS a wavefront takes, and so how many a CU holds)
    go(width <= 4u ? beam_kernel<4> : width <= 16u ? beam_kernel<16> : beam_kernel<kBeamMaxWidth>,
       (unsigned)batch->n, kBlock, *batch, l, ws, call);
    for (uint32_t m = 1; m <= batch->max_chunks; ++m, half ^= 1) {
      go(beam_eval_kernel<true, true, true>, blocks_for(lanes), kBlock, *batch, l, ws, m, half, call);
      go(beam_select_kernel<true>, (unsigned)batch->n, kBlock, *batch, l, ws, m, half, call);
    }
  } else {
    go(beam_init_kernel, per_scenario, 256, *batch, l, ws);
    for (uint32_t m = 1; m <= batch->max_chunks; ++m, half ^= 1) {
      go(fix ? beam_eval_kernel<false, true, false> : beam_eval_kernel<false, false, false>,
         blocks_for(lanes), kBlock, *batch, l, ws, m, half, 0ull);
      go(beam_eval_kernel<true, true, false>, blocks_for(lanes), kBlock, *batch, l, ws, m, half, 0ull);
      go(beam_select_kernel<false>, (unsigned)batch->n, kBlock, *batch, l, ws, m, half, 0ull);
    }
  }
  go(beam_finish_kernel, per_scenario, 256, *batch, l, (const uint8_t*)ws, best_t, best_orders);
  return go.status();
}

int themis_metrics_batch(const themis_batch_t* batch, const double* t_done, const double* transfer,
                         double* utilization, double* ideal, void* stream) {
  if (!batch) return THEMIS_ERR_INVALID_ARGUMENT;
  if (batch->n == 0) return THEMIS_OK;
  if (!batch->ndims || !batch->bw || !t_done || !transfer) return THEMIS_ERR_INVALID_ARGUMENT;
  if (batch->n_coll ? !batch->coll_size : !batch->size_bytes) return THEMIS_ERR_INVALID_ARGUMENT;
  if (batch->n > (uint64_t)0x7fffffff * 256u) return THEMIS_ERR_UNSUPPORTED;
  Launcher go(stream);
  go(metrics_kernel, (unsigned)((batch->n + 255) / 256), 256, *batch, t_done, transfer,
     utilization, ideal);
  return go.status();
}

int themis_classify_batch(const themis_batch_t* batch, uint8_t* classes, void* stream) {
  if (!batch) return THEMIS_ERR_INVALID_ARGUMENT;
  if (batch->n == 0) return THEMIS_OK;
  if (!batch->ndims || !batch->npus || !batch->bw || !classes) return THEMIS_ERR_INVALID_ARGUMENT;
  if (batch->n > (uint64_t)0x7fffffff * 256u) return THEMIS_ERR_UNSUPPORTED;
  Launcher go(stream);
  go(classify_kernel, (unsigned)((batch->n + 255) / 256), 256, *batch, classes);
  return go.status();
}

int themis_sweep_best(uint64_t n, int n_thr, int n_pol, const double* t_done, int baseline_col,
                      double* best_t, uint32_t* best_thr, double* speedup, void* stream) {
  if (n_thr < 1 || n_pol < 1 || n_pol > 3 || baseline_col >= n_pol) return THEMIS_ERR_INVALID_ARGUMENT;
  if (n == 0) return THEMIS_OK;
  if (!t_done || !best_t) return THEMIS_ERR_INVALID_ARGUMENT;
  if (n > (uint64_t)0x7fffffff * 64u) return THEMIS_ERR_UNSUPPORTED;
  const uint64_t items = n * (uint64_t)n_pol;
  Launcher go(stream);
  go(sweep_best_kernel, (unsigned)((items + 255) / 256), 256, n, (uint32_t)n_thr, (uint32_t)n_pol,
     t_done, baseline_col, best_t, best_thr, speedup);
  return go.status();
}

}  // extern "C"
