// Planner and queue simulation with a whole wavefront per evaluation, for
// batches too small to fill the GPU with one lane per scenario, and for NPU
// counts that are not powers of two.
//
// With one lane per scenario the time of a small batch is the time of one
// lane's chain of events: every event pays the instructions of all the
// branches that some lane of the wavefront takes, the selects among the four
// dimensions' registers, and three dependent LDS round trips.  Here all
// control flow is the same for the 64 lanes: which stage ends, which list a
// chunk joins and which one is served are scalar values, so an event executes
// only what it needs, and the lanes of a register serve as memory that a
// scalar index reaches in one instruction (v_readlane / v_writelane) instead
// of an LDS round trip:
//   * what depends on a chunk's order alone (stage times, what a completion
//     does) sits in per-dimension tables, lane = rank of the order + 24 * phase
//     (48 lanes for the 24 orders of four dimensions).  Their entries are made
//     by the step-by-step arithmetic of the model (divisions by P_k), so any
//     NPU counts are covered and the results are those of the other paths to
//     the last bit;
//   * queues: first-in-first-out keeps a ring per dimension; Smallest-Chunk-
//     First a list per (dimension, size class), head and tail in lane = class,
//     links in lane = chunk.  The sizes that can wait for one dimension are at
//     most 48 (24 orders, two phases), so a 64-bit scalar per dimension says
//     which lists hold chunks.  Chunks that wait for their first stage are
//     taken from an array in chunk order: their size is the largest there is
//     (the smallest, for a stand-alone All-Gather), so they come after (before)
//     all lists.
// An event is some 60 scalar and vector instructions and, up to 64 chunks, no
// memory access (beyond them the links and part of the queues are in LDS, and
// where the records are asked for 64 of them go there at a time).
#pragma once

#include "themis_generic.hpp"
#include "themis_ring.hpp"

namespace themis {

// Value of lane `lane` (the same for all lanes) of v, and v with that lane replaced.
__device__ __forceinline__ uint32_t lane_get(uint32_t v, uint32_t lane) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)lane);
}
// (clang has no builtin for v_writelane)
extern "C" __device__ int themis_write_lane(int value, int lane, int old) __asm("llvm.amdgcn.writelane.i32");
__device__ __forceinline__ uint32_t lane_put(uint32_t v, uint32_t lane, uint32_t x) {
  return (uint32_t)themis_write_lane((int)x, (int)lane, (int)v);
}
__device__ __forceinline__ double lane_get(double v, uint32_t lane) {
  return __hiloint2double((int)lane_get((uint32_t)__double2hiint(v), lane),
                          (int)lane_get((uint32_t)__double2loint(v), lane));
}
__device__ __forceinline__ uint32_t first_lane(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}
// A condition on values that are the same in all lanes, as a scalar.
__device__ __forceinline__ bool uniform(bool c) { return __builtin_amdgcn_ballot_w64(c) != 0ull; }
// its outcome as the given bit(s)
__device__ __forceinline__ uint32_t uniform_bit(bool c, uint32_t bit) {
  return (uint32_t)__builtin_amdgcn_ballot_w64(c) & bit;
}
__device__ __forceinline__ uint32_t lane_id() { return threadIdx.x & 63u; }

// ---------------------------------------------------------------------------
// Planner (Alg. 1): lane = outcome of the six comparisons of the loads (see
// plan_order_entry).  The table holds, per outcome, the order code, the
// threshold of the dimension that is then the least loaded, and what a chunk
// of that order adds to each dimension's load; a chunk is six comparisons and
// a few lane reads (one lane per scenario: some 900 clocks per chunk on a lone
// wavefront, here about 250).
// ---------------------------------------------------------------------------
template <uint32_t kDims, typename Flush>
__device__ __forceinline__ void wave_plan_chunks(uint32_t C, bool themis, double thr, uint32_t code,
                                                 const double (&inc)[kMaxDims],
                                                 double (&load)[kMaxDims], Flush flush) {
  uint32_t acc = ~0u;
  for (uint32_t c = 0; c < C; ++c) {
    uint32_t outcome = 0u;
    if (kDims > 1u && themis) {
      double lo = load[0], hi = load[0];
#pragma unroll
      for (uint32_t k = 1; k < kDims; ++k) {
        lo = min_f64(lo, load[k]);
        hi = -min_f64(-hi, -load[k]);
      }
      uint32_t bit = 1u;
#pragma unroll
      for (uint32_t a = 0; a < (uint32_t)kMaxDims; ++a)
#pragma unroll
        for (uint32_t b = a + 1u; b < (uint32_t)kMaxDims; ++b, bit <<= 1)
          if (b < kDims) outcome |= uniform_bit(load[a] > load[b], bit);
      if (uniform((hi - lo) < lane_get(thr, outcome))) outcome = 0u;
    }
    acc = lane_put(acc, c & 63u, lane_get(code, outcome));
#pragma unroll
    for (uint32_t k = 0; k < kDims; ++k) load[k] = load[k] + lane_get(inc[k], outcome);
    if ((c & 63u) == 63u) flush(c - 63u, acc);
  }
  if (C & 63u) flush(C & ~63u, acc);
}

// flush(first, codes): lane L holds the order code of chunk first + L.
template <typename Flush>
__device__ __forceinline__ void wave_plan(const Scenario& s, double chunk, bool themis, bool rel,
                                          double thr_in, double (&load)[kMaxDims], Flush flush) {
  const uint32_t D = (uint32_t)s.D;
  const bool gather = s.ctype == THEMIS_COLL_ALL_GATHER;
  const bool twice = s.ctype == THEMIS_COLL_ALL_REDUCE;
  // the lane's own outcome: the dimensions in ascending order of the loads
  // (unused dimensions are never before a used one: no comparison with them is set)
  const uint32_t o = lane_id();
  const uint32_t a01 = o & 1u, a02 = (o >> 1) & 1u, a03 = (o >> 2) & 1u;
  const uint32_t a12 = (o >> 3) & 1u, a13 = (o >> 4) & 1u, a23 = (o >> 5) & 1u;
  const uint32_t r1 = (1u - a01) + a12 + a13, r2 = (1u - a02) + (1u - a12) + a23;
  const uint32_t r3 = (1u - a03) + (1u - a13) + (1u - a23);
  uint32_t code = ((1u << (2u * r1)) | (2u << (2u * r2)) | (3u << (2u * r3))) & 0xffu;
  code &= (1u << (2u * D)) - 1u;
  double thr = thr_in;
  if (rel) {
    const int kmin = (int)(code & 3u);
    const double cmin = sel4(kmin, s.coef[0], s.coef[1], s.coef[2], s.coef[3]);
    double whole = chunk;
    if (gather) whole = chunk * (double)sel4(kmin, s.P[0], s.P[1], s.P[2], s.P[3]);
    thr = thr_in * (whole * cmin);
  }
  if (gather) code = reverse_code(code, (int)D);
  double inc[kMaxDims] = {0.0, 0.0, 0.0, 0.0};
  double x = chunk;
  for (uint32_t j = 0; j < D; ++j) {
    const int k = (int)((code >> (2u * j)) & 3u);
    const double ck = sel4(k, s.coef[0], s.coef[1], s.coef[2], s.coef[3]);
    const double pk = (double)sel4(k, s.P[0], s.P[1], s.P[2], s.P[3]);
    if (gather) x = x * pk;
    const double t = x * ck;
    const double add = twice ? t + t : t;
#pragma unroll
    for (int kk = 0; kk < kMaxDims; ++kk)
      if (kk == k) inc[kk] = add;
    if (!gather) x = x / pk;
  }
#pragma unroll
  for (uint32_t k = 0; k < (uint32_t)kMaxDims; ++k)
    load[k] = k < D ? tracker_start(s, (int)k) : 0.0;
  switch (D) {
    case 1: wave_plan_chunks<1>(s.C, themis, thr, code, inc, load, flush); break;
    case 2: wave_plan_chunks<2>(s.C, themis, thr, code, inc, load, flush); break;
    case 3: wave_plan_chunks<3>(s.C, themis, thr, code, inc, load, flush); break;
    default: wave_plan_chunks<4>(s.C, themis, thr, code, inc, load, flush); break;
  }
}

// ---------------------------------------------------------------------------
// Queue simulation.
// ---------------------------------------------------------------------------
constexpr uint32_t kWaveOrders = 24u;
constexpr uint32_t kWaveIdMask = 0x1ffu;      // chunk id: bits 0-8 of a record
constexpr uint32_t kWaveStateShift = 9u;      // order rank + 24 * phase: bits 9-14
constexpr uint32_t kWaveFinished = 1u << 15;  // (of a running stage only)
constexpr uint32_t kWaveClassShift = 16u;     // list the chunk joins then: class bits 16-21,
constexpr uint32_t kWaveDimShift = 22u;       // dimension bits 22-23
constexpr uint32_t kWaveTurned = 1u << 24;    // (of a table's entry) the stage and the one after it, see QuadStages

// Per-order tables of one evaluation, lane = order rank + 24 * phase.
struct WaveTables {
  double time[kMaxDims];     // stage time on dimension k
  uint32_t next[kMaxDims];   // what the completion there does: state, finished, class, dimension
  double t_min;              // smallest stage time of any order in use (all lanes)
  bool normal;               // no size leaves the normal range (all lanes)
  uint32_t first_class[kMaxDims];  // class of a chunk before its first stage, on dimension k
  bool few_classes;          // at most 16 classes on every dimension (all lanes)
};

// orders_used: bit r says that some chunk has the order of rank r.  turns: with kWaveTurned.
__device__ __forceinline__ void wave_tables(const Scenario& s, double chunk, bool scf,
                                            uint32_t orders_used, WaveTables& t, bool turns) {
  const uint32_t D = (uint32_t)s.D;
  const bool rs_only = s.ctype == THEMIS_COLL_REDUCE_SCATTER;
  const bool gather = s.ctype == THEMIS_COLL_ALL_GATHER;
  const uint32_t lane = lane_id();
  const uint32_t phase = lane >= kWaveOrders ? 1u : 0u;
  const uint32_t rank = lane - (phase ? kWaveOrders : 0u);
  const bool valid = lane < 2u * kWaveOrders && ((orders_used >> (rank & 31u)) & 1u) != 0u &&
                     (phase ? !rs_only : !gather);
  const uint32_t code = ring_order_of_rank(rank < kWaveOrders ? rank : 0u);
  double before_rs[kMaxDims], before_ag[kMaxDims];
  uint32_t place[kMaxDims];   // of dimension k in the order
#pragma unroll
  for (int k = 0; k < kMaxDims; ++k) {
    t.time[k] = 0.0;
    before_rs[k] = before_ag[k] = 0.0;
    place[k] = 0u;
  }
  double x = chunk, smallest = chunk, largest = chunk, tmin = inf64();
  // Reduce-Scatter stages shrink the resident size, one division at a time
  for (uint32_t j = 0; j < D; ++j) {
    const int kj = (int)((code >> (2u * j)) & 3u);
    const double time = x * sel4(kj, s.coef[0], s.coef[1], s.coef[2], s.coef[3]);
#pragma unroll
    for (int k = 0; k < kMaxDims; ++k)
      if (k == kj) { place[k] = j; before_rs[k] = x; t.time[k] = time; }
    if (!gather) {
      x = x / (double)sel4(kj, s.P[0], s.P[1], s.P[2], s.P[3]);
      smallest = min_f64(smallest, x);
    }
  }
  // All-Gather stages grow it (back), last field first; a stand-alone
  // All-Gather moves the grown size, one that follows a Reduce-Scatter takes
  // that one's time
  for (uint32_t j = D; j-- > 0u;) {
    const int kj = (int)((code >> (2u * j)) & 3u);
    const double size = x;
    x = x * (double)sel4(kj, s.P[0], s.P[1], s.P[2], s.P[3]);
    largest = -min_f64(-largest, -x);
    const double time = x * sel4(kj, s.coef[0], s.coef[1], s.coef[2], s.coef[3]);
#pragma unroll
    for (int k = 0; k < kMaxDims; ++k)
      if (k == kj) { before_ag[k] = size; t.time[k] = gather ? time : t.time[k]; }
  }
  const bool in_range = smallest >= 2.2250738585072014e-308 && largest < inf64();
  uint32_t cls[kMaxDims] = {0u, 0u, 0u, 0u};
  const uint64_t rows = __builtin_amdgcn_ballot_w64(valid);
  t.normal = __builtin_amdgcn_ballot_w64(valid && !in_range) == 0ull;
#pragma unroll
  for (int k = 0; k < kMaxDims; ++k) {
    if (k < (int)D) {
      if (s.has_fix) t.time[k] = s.fix[k] + t.time[k];
      tmin = min_f64(tmin, t.time[k]);
      if (scf) {
        const double v = phase ? before_ag[k] : before_rs[k];
        // one step per distinct size
        for (uint64_t m = rows; m != 0ull;) {
          const double one = lane_get(v, (uint32_t)__builtin_ctzll(m));
          cls[k] += one < v ? 1u : 0u;
          m &= ~__builtin_amdgcn_ballot_w64(one == v);
        }
      }
    }
  }
  t.few_classes = __builtin_amdgcn_ballot_w64(valid && (cls[0] | cls[1] | cls[2] | cls[3]) > 15u) == 0ull;
#pragma unroll
  for (int k = 0; k < kMaxDims; ++k) t.first_class[k] = cls[k];
  if (!valid) tmin = inf64();
  for (int off = 32; off > 0; off >>= 1) tmin = min_f64(tmin, __shfl_xor(tmin, off));
  t.t_min = tmin;
#pragma unroll
  for (int k = 0; k < kMaxDims; ++k) {
    const uint32_t p = place[k];
    const uint32_t turned = (uint32_t)__shfl((int)cls[k], (int)((lane + kWaveOrders) & 63u));
    uint32_t kn, c, ph = phase;
    bool fin;
    if (phase == 0u && p + 1u == D) {   // the last Reduce-Scatter: the All-Gather starts on k itself
      fin = rs_only;
      kn = (uint32_t)k;
      c = turned;
      ph = 1u;
    } else {
      const uint32_t at = phase ? p - 1u : p + 1u;
      fin = phase != 0u && p == 0u;
      kn = (code >> ((2u * at) & 31u)) & 3u;
      c = sel4((int)kn, cls[0], cls[1], cls[2], cls[3]);
    }
    t.next[k] = ((rank + kWaveOrders * ph) & 63u) << kWaveStateShift | (fin ? kWaveFinished : 0u) |
                (c & 63u) << kWaveClassShift | kn << kWaveDimShift;
    // Smallest-Chunk-First: the last Reduce-Scatter and the All-Gather that follows it at once
    // (same dimension, same time, no smaller chunk waits) are one stage of twice the time
    if (turns && scf && !rs_only) {
      const uint32_t after = (uint32_t)__shfl((int)t.next[k], (int)((lane + kWaveOrders) & 63u));
      if (phase == 0u && p + 1u == D) t.next[k] = after | kWaveTurned;
    }
  }
}

// One dimension of the event loop.
struct WaveDim {
  double finish, busy;        // of the running stage (quiet NaN: idle); service time so far
  uint32_t running;           // chunk and next state, what its completion does
  uint32_t started;           // operations so far
  uint32_t queue;             // lane = place & 63: the ring (FIFO), else the chunks that wait
                              // for their first stage, in chunk order; beyond 64 chunks the
                              // block of 64 places that holds place `get`, the rest in LDS
  uint32_t get, put;          // places taken and filled so far
  uint64_t lists;             // bit c: list of class c holds chunks
  uint32_t head, tail;        // lane = class: records of its first and last chunk
  uint32_t log;               // lane = operation number & 63: the last records started
};

// LDS of one evaluation while the event loop runs.
template <uint32_t kWords>
struct WaveLds {
  static constexpr uint32_t kCap = 64u * kWords;
  uint16_t queue[kMaxDims][kCap];       // the chunks that start on each dimension / the rings
  uint16_t link[kCap];                  // (beyond 64 chunks) next chunk of its list
  uint16_t log[kMaxDims][2u * kCap];    // records in the order each dimension executed them
};

// The event loop is one assembly block.  Written in C++ it comes out with its
// scalar control flow turned into copies of some forty registers per branch
// (353 us for the six platforms of Table 2 at 64 chunks, 24 scenarios, where
// this loop takes a fifth), and what makes the mapping pay is that an event is
// only the instructions below.
//
// Operands, K = dimension:  fK finish, zK busy, aK / bK low and high half of the
// stage times, nK table of completions, hK / lK head and tail, qK queue, gK
// log; scalars rK running, xK lists, iK / oK places taken / filled, cK started.
// lk: links, now: clock, idle: bits of idle dimensions.
//
// Wait states the hardware does not insert here (gfx950): a scalar written by a
// vector instruction is read by another vector instruction two instructions
// later at the earliest, and serves as lane select only after a scalar
// instruction has rewritten it; a vector register is read by v_readlane one
// instruction after it was written at the earliest.
//
// The stage of record rc starts on K.  E, X: label suffix.
#define THEMIS_W_LOG_0(K)
#define THEMIS_W_LOG_1(K) "v_writelane_b32 %[g" #K "], %[rc], m0\n\t"
#define THEMIS_W_FLUSH(K, E) \
  "s_and_b32 %[t], %[c" #K "], 63\n\t" "s_cbranch_scc0 .Lwf" #E "_%=\n\t" ".Lwg" #E "_%=:\n\t"
#define THEMIS_W_START(K, E, LOG, P)                                                  \
  "s_lshr_b32 %[t], %[rc], 9\n\t"                                                     \
  "s_mov_b32 m0, %[c" #K "]\n\t"                                                      \
  "v_readlane_b32 vcc_lo, %[a" #K "], %[t]\n\t"                                       \
  "v_readlane_b32 vcc_hi, %[b" #K "], %[t]\n\t"                                       \
  "v_readlane_b32 %[nx], %[n" #K "], %[t]\n\t"                                        \
  "s_and_b32 %[t], %[rc], 0x1ff\n\t" THEMIS_W_LOG_##LOG(K)                            \
  "s_add_u32 %[c" #K "], %[c" #K "], 1\n\t"                                           \
  "v_add_f64 %[f" #K "], %[now], vcc\n\t"                                             \
  "v_add_f64 %[z" #K "], %[z" #K "], vcc\n\t"                                         \
  "s_or_b32 %[r" #K "], %[t], %[nx]\n\t"                                              \
  "s_bitset0_b32 %[idle], " #K "\n\t" THEMIS_W_FLUSH(K, E) THEMIS_W_TURN_##P(K, E)
// the stage is two (kWaveTurned): the second one out of line
#define THEMIS_W_TURN_FIFO1(K, E)
#define THEMIS_W_TURN_FIFO2(K, E)
#define THEMIS_W_TURN_SCF1(K, E) \
  "s_bitcmp1_b32 %[r" #K "], 24\n\t" "s_cbranch_scc1 .Lwu" #E "_%=\n\t" ".Lwv" #E "_%=:\n\t"
#define THEMIS_W_TURN_SCF2(K, E) THEMIS_W_TURN_SCF1(K, E)
#define THEMIS_W_TURN_AWAY_FIFO1(K, E, LOG)
#define THEMIS_W_TURN_AWAY_FIFO2(K, E, LOG)
#define THEMIS_W_TURN_AWAY_SCF1(K, E, LOG)                                            \
  ".Lwu" #E "_%=:\n\t" "s_mov_b32 m0, %[c" #K "]\n\t" "s_bitset0_b32 %[r" #K "], 24\n\t" \
  "v_add_f64 %[f" #K "], %[f" #K "], vcc\n\t" "v_add_f64 %[z" #K "], %[z" #K "], vcc\n\t" \
  "s_add_u32 %[rc], %[rc], 24*512\n\t" "s_add_u32 %[c" #K "], %[c" #K "], 1\n\t" "s_nop 1\n\t" \
  THEMIS_W_LOG_##LOG(K)                                                               \
  "s_and_b32 %[t], %[c" #K "], 63\n\t" "s_cbranch_scc1 .Lwv" #E "_%=\n\t"             \
  "s_cmp_gt_u32 %[c" #K "], %[most]\n\t" "s_cbranch_scc1 .Lwend_%=\n\t"               \
  THEMIS_W_STORE_##LOG(K) "s_branch .Lwv" #E "_%=\n\t"
#define THEMIS_W_TURN_AWAY_SCF2(K, E, LOG) THEMIS_W_TURN_AWAY_SCF1(K, E, LOG)
// out of line, every 64 operations of the dimension: the end of a loop whose
// records are broken, else 64 records of the log to LDS (rb: bytes of a
// dimension's log)
#define THEMIS_W_STORE_0(K)
#define THEMIS_W_STORE_1(K)                                                           \
  "s_mul_i32 %[nx], %[rb], " #K "\n\t" "s_lshl1_add_u32 %[t], %[c" #K "], %[nx]\n\t" \
  "v_add_u32_e32 %[va], %[t], %[logat]\n\t" "ds_write_b16 %[va], %[g" #K "]\n\t"
#define THEMIS_W_START_AWAY(K, E, LOG, P)                                             \
  ".Lwf" #E "_%=:\n\t" "s_cmp_gt_u32 %[c" #K "], %[most]\n\t" "s_cbranch_scc1 .Lwend_%=\n\t" \
  THEMIS_W_STORE_##LOG(K) "s_branch .Lwg" #E "_%=\n\t" THEMIS_W_TURN_AWAY_##P(K, E, LOG)

// --- first-in-first-out, up to 64 chunks: the ring is a register
#define THEMIS_W_PUSH_FIFO1(N, E)                                                     \
  "s_mov_b32 m0, %[o" #N "]\n\t" "s_add_u32 %[o" #N "], %[o" #N "], 1\n\t"            \
  "v_writelane_b32 %[q" #N "], %[rc], m0\n\t"
#define THEMIS_W_PUSH_AWAY_FIFO1(N, E)
#define THEMIS_W_PICK_FIFO1(K, E, DONE, LOG)                                          \
  "s_cmp_eq_u32 %[i" #K "], %[o" #K "]\n\t" "s_cbranch_scc1 " DONE "\n\t"             \
  "v_readlane_b32 %[rc], %[q" #K "], %[i" #K "]\n\t"                                  \
  "s_add_u32 %[i" #K "], %[i" #K "], 1\n\t" THEMIS_W_START(K, E, LOG, FIFO1)
#define THEMIS_W_PICK_AWAY_FIFO1(K, E, DONE, LOG) THEMIS_W_START_AWAY(K, E, LOG, FIFO1)

// --- beyond 64 chunks: the ring in LDS, the block that is being taken from
// also in the register
#define THEMIS_W_PUSH_FIFO2(N, E)                                                     \
  "s_and_b32 %[t], %[o" #N "], %[cap]-1\n\t"                                          \
  "v_mov_b32_e32 %[vd], %[rc]\n\t"                                                    \
  "s_lshl1_add_u32 %[t], %[t], %[queueat]\n\t"                                        \
  "s_mov_b32 m0, %[o" #N "]\n\t"                                                      \
  "v_mov_b32_e32 %[va], %[t]\n\t"                                                     \
  "s_mov_b64 exec, 1\n\t" "ds_write_b16 %[va], %[vd] offset:%[cap]*2*" #N "\n\t"      \
  "s_mov_b64 exec, -1\n\t"                                                            \
  "s_xor_b32 %[t], %[o" #N "], %[i" #N "]\n\t" "s_add_u32 %[o" #N "], %[o" #N "], 1\n\t" \
  "s_cmp_gt_u32 %[t], 63\n\t" "s_cbranch_scc1 .Lwp" #E "_%=\n\t"                      \
  "v_writelane_b32 %[q" #N "], %[rc], m0\n\t" ".Lwp" #E "_%=:\n\t"
#define THEMIS_W_PUSH_AWAY_FIFO2(N, E)
#define THEMIS_W_PICK_FIFO2(K, E, DONE, LOG)                                          \
  "s_cmp_eq_u32 %[i" #K "], %[o" #K "]\n\t" "s_cbranch_scc1 " DONE "\n\t"             \
  "v_readlane_b32 %[rc], %[q" #K "], %[i" #K "]\n\t"                                  \
  "s_add_u32 %[i" #K "], %[i" #K "], 1\n\t"                                           \
  "s_and_b32 %[t], %[i" #K "], 63\n\t" "s_cbranch_scc0 .Lwr" #E "_%=\n\t"             \
  ".Lws" #E "_%=:\n\t" THEMIS_W_START(K, E, LOG, FIFO2)
#define THEMIS_W_RELOAD(K, E)                                                         \
  ".Lwr" #E "_%=:\n\t" "s_and_b32 %[t], %[i" #K "], %[cap]-1\n\t" "s_lshl_b32 %[t], %[t], 1\n\t" \
  "v_add_u32_e32 %[va], %[t], %[queuelane]\n\t"                                       \
  "ds_read_u16 %[q" #K "], %[va] offset:%[cap]*2*" #K "\n\t" "s_waitcnt lgkmcnt(0)\n\t" \
  "s_branch .Lws" #E "_%=\n\t"
#define THEMIS_W_PICK_AWAY_FIFO2(K, E, DONE, LOG) THEMIS_W_RELOAD(K, E) THEMIS_W_START_AWAY(K, E, LOG, FIFO2)

// --- Smallest-Chunk-First, up to 64 chunks: links in lane = chunk
#define THEMIS_W_PUSH_SCF1(N, E)                                                      \
  "s_bfe_u32 %[c], %[rn], 0x60010\n\t"                                                \
  "s_bitcmp1_b64 %[x" #N "], %[c]\n\t" "s_cbranch_scc0 .Lwe" #E "_%=\n\t"             \
  "v_readlane_b32 %[t], %[l" #N "], %[c]\n\t" "s_and_b32 %[t], %[t], 0x1ff\n\t"       \
  "s_mov_b32 m0, %[t]\n\t" "s_nop 0\n\t" "v_writelane_b32 %[lk], %[rc], m0\n\t"       \
  "s_mov_b32 m0, %[c]\n\t" "s_nop 0\n\t" "v_writelane_b32 %[l" #N "], %[rc], m0\n\t"  \
  ".Lwp" #E "_%=:\n\t"
#define THEMIS_W_PUSH_AWAY_SCF1(N, E)                                                 \
  ".Lwe" #E "_%=:\n\t" "s_mov_b32 m0, %[c]\n\t" "s_bitset1_b64 %[x" #N "], %[c]\n\t"  \
  "v_writelane_b32 %[h" #N "], %[rc], m0\n\t" "v_writelane_b32 %[l" #N "], %[rc], m0\n\t" \
  "s_branch .Lwp" #E "_%=\n\t"
#define THEMIS_W_PICK_SCF1(K, E, DONE, LOG)                                           \
  "s_cmp_eq_u64 %[x" #K "], 0\n\t" "s_cbranch_scc1 .Lwi" #E "_%=\n\t"                 \
  "s_ff1_i32_b64 %[c], %[x" #K "]\n\t"                                                \
  "v_readlane_b32 %[rc], %[h" #K "], %[c]\n\t"                                        \
  "v_readlane_b32 %[nx], %[l" #K "], %[c]\n\t"                                        \
  "s_and_b32 %[t], %[rc], 0x1ff\n\t" "s_mov_b32 m0, %[c]\n\t"                         \
  "v_readlane_b32 %[t], %[lk], %[t]\n\t"                                              \
  "s_cmp_eq_u32 %[rc], %[nx]\n\t" "s_cselect_b32 %[nx], 1, 0\n\t"                     \
  "s_bfm_b64 vcc, %[nx], %[c]\n\t" "s_xor_b64 %[x" #K "], %[x" #K "], vcc\n\t"        \
  "v_writelane_b32 %[h" #K "], %[t], m0\n\t" ".Lws" #E "_%=:\n\t" THEMIS_W_START(K, E, LOG, SCF1)
#define THEMIS_W_PICK_AWAY_SCF1(K, E, DONE, LOG)                                      \
  ".Lwi" #E "_%=:\n\t" "s_cmp_eq_u32 %[i" #K "], %[o" #K "]\n\t" "s_cbranch_scc1 " DONE "\n\t" \
  "v_readlane_b32 %[rc], %[q" #K "], %[i" #K "]\n\t" "s_add_u32 %[i" #K "], %[i" #K "], 1\n\t" \
  "s_branch .Lws" #E "_%=\n\t" THEMIS_W_START_AWAY(K, E, LOG, SCF1)

// --- beyond 64 chunks: links in LDS; the link of the chunk taken is on its way
// while its stage starts
#define THEMIS_W_PUSH_SCF2(N, E)                                                      \
  "s_bfe_u32 %[c], %[rn], 0x60010\n\t"                                                \
  "s_bitcmp1_b64 %[x" #N "], %[c]\n\t" "s_cbranch_scc0 .Lwe" #E "_%=\n\t"             \
  "v_readlane_b32 %[t], %[l" #N "], %[c]\n\t" "s_and_b32 %[t], %[t], 0x1ff\n\t"       \
  "v_mov_b32_e32 %[vd], %[rc]\n\t"                                                    \
  "s_lshl1_add_u32 %[t], %[t], %[linkat]\n\t" "s_mov_b32 m0, %[c]\n\t"                \
  "v_mov_b32_e32 %[va], %[t]\n\t"                                                     \
  "s_mov_b64 exec, 1\n\t" "ds_write_b16 %[va], %[vd]\n\t" "s_mov_b64 exec, -1\n\t"    \
  "v_writelane_b32 %[l" #N "], %[rc], m0\n\t" ".Lwp" #E "_%=:\n\t"
#define THEMIS_W_PUSH_AWAY_SCF2(N, E) THEMIS_W_PUSH_AWAY_SCF1(N, E)
#define THEMIS_W_PICK_SCF2(K, E, DONE, LOG)                                           \
  "s_cmp_eq_u64 %[x" #K "], 0\n\t" "s_cbranch_scc1 .Lwi" #E "_%=\n\t"                 \
  "s_ff1_i32_b64 %[c], %[x" #K "]\n\t"                                                \
  "v_readlane_b32 %[rc], %[h" #K "], %[c]\n\t"                                        \
  "v_readlane_b32 %[nx], %[l" #K "], %[c]\n\t"                                        \
  "s_and_b32 %[t], %[rc], 0x1ff\n\t" "s_lshl1_add_u32 %[t], %[t], %[linkat]\n\t"      \
  "v_mov_b32_e32 %[va], %[t]\n\t" "ds_read_u16 %[vd], %[va]\n\t"                      \
  "s_cmp_eq_u32 %[rc], %[nx]\n\t" "s_cselect_b32 %[nx], 1, 0\n\t"                     \
  "s_bfm_b64 vcc, %[nx], %[c]\n\t" "s_xor_b64 %[x" #K "], %[x" #K "], vcc\n\t"        \
  THEMIS_W_START(K, E, LOG, SCF2)                                                           \
  "s_waitcnt lgkmcnt(0)\n\t" "s_mov_b32 m0, %[c]\n\t"                                 \
  "v_readfirstlane_b32 %[t], %[vd]\n\t" "s_nop 1\n\t"                                 \
  "v_writelane_b32 %[h" #K "], %[t], m0\n\t"
#define THEMIS_W_PICK_AWAY_SCF2(K, E, DONE, LOG)                                      \
  ".Lwi" #E "_%=:\n\t" "s_cmp_eq_u32 %[i" #K "], %[o" #K "]\n\t" "s_cbranch_scc1 " DONE "\n\t" \
  "v_readlane_b32 %[rc], %[q" #K "], %[i" #K "]\n\t" "s_add_u32 %[i" #K "], %[i" #K "], 1\n\t" \
  "s_and_b32 %[t], %[i" #K "], 63\n\t" "s_cbranch_scc0 .Lwr" #E "_%=\n\t"             \
  ".Lws" #E "_%=:\n\t" THEMIS_W_START(K, E##i, LOG, SCF2) "s_branch " DONE "\n\t"           \
  THEMIS_W_RELOAD(K, E) THEMIS_W_START_AWAY(K, E, LOG, SCF2) THEMIS_W_START_AWAY(K, E##i, LOG, SCF2)

// The stage that has ended on K (one completion at this instant): its chunk
// joins its next list, or starts at once where that dimension is idle; then K
// takes its next chunk.
#define THEMIS_W_HAND_ON(K, N, P, LOG)                                                \
  "s_bitcmp1_b32 %[idle], " #N "\n\t" "s_cbranch_scc1 .Lwd" #K #N "_%=\n\t"           \
  THEMIS_W_PUSH_##P(N, K##N) "s_branch .Lwk" #K "_%=\n\t"
// (in front of what only branches lead to: at the start of a 32-byte line; 50 first-in-first-out
// scenarios of 64 chunks 118 -> 115.7 us)
#define THEMIS_W_LINE ".p2align 5\n\t"
#define THEMIS_W_HAND_ON_AWAY(K, N, P, LOG)                                           \
  THEMIS_W_PUSH_AWAY_##P(N, K##N)                                                     \
  THEMIS_W_LINE ".Lwd" #K #N "_%=:\n\t" THEMIS_W_START(N, d##K##N, LOG, P) "s_branch .Lwk" #K "_%=\n\t" \
  THEMIS_W_START_AWAY(N, d##K##N, LOG, P)
// A, B, C: the other dimensions
#define THEMIS_W_ENDED(K, A, B, C, P, LOG)                                            \
  ".Lwc" #K "_%=:\n\t"                                                                \
  "s_mov_b32 %[rn], %[r" #K "]\n\t" "v_mov_b64_e32 %[f" #K "], %[nan]\n\t"            \
  "s_and_b32 %[rc], %[rn], 0x7fff\n\t"                                                \
  "s_bitcmp1_b32 %[rn], 15\n\t" "s_cbranch_scc1 .Lwl" #K "_%=\n\t"                    \
  "s_lshr_b32 %[t], %[rn], 22\n\t"                                                    \
  "s_cmp_eq_u32 %[t], " #A "\n\t" "s_cbranch_scc1 .Lwt" #K #A "_%=\n\t"               \
  "s_cmp_eq_u32 %[t], " #B "\n\t" "s_cbranch_scc1 .Lwt" #K #B "_%=\n\t"               \
  "s_cmp_eq_u32 %[t], " #C "\n\t" "s_cbranch_scc1 .Lwt" #K #C "_%=\n\t"               \
  THEMIS_W_PUSH_##P(K, K##K)                                                          \
  ".Lwl" #K "_%=:\n\t" "s_bitset1_b32 %[idle], " #K "\n\t"                            \
  ".Lwk" #K "_%=:\n\t" THEMIS_W_PICK_##P(K, K, ".Lwnext_%=", LOG) "s_branch .Lwnext_%=\n\t" \
  THEMIS_W_LINE ".Lwt" #K #A "_%=:\n\t" "s_bitset1_b32 %[idle], " #K "\n\t" THEMIS_W_HAND_ON(K, A, P, LOG) \
  THEMIS_W_LINE ".Lwt" #K #B "_%=:\n\t" "s_bitset1_b32 %[idle], " #K "\n\t" THEMIS_W_HAND_ON(K, B, P, LOG) \
  THEMIS_W_LINE ".Lwt" #K #C "_%=:\n\t" "s_bitset1_b32 %[idle], " #K "\n\t" THEMIS_W_HAND_ON(K, C, P, LOG) \
  THEMIS_W_PUSH_AWAY_##P(K, K##K) THEMIS_W_PICK_AWAY_##P(K, K, ".Lwnext_%=", LOG)     \
  THEMIS_W_HAND_ON_AWAY(K, A, P, LOG) THEMIS_W_HAND_ON_AWAY(K, B, P, LOG)             \
  THEMIS_W_HAND_ON_AWAY(K, C, P, LOG)

// Several completions at one instant: handed on one by one, the lowest chunk id
// first, so that equal arrival times are appended in chunk-id order; then every
// idle dimension takes its next chunk.
#define THEMIS_W_LOWEST(K)                                                            \
  "s_and_b32 %[t], %[r" #K "], 0x1ff\n\t" "s_bitcmp1_b32 %[ends], " #K "\n\t"         \
  "s_cselect_b32 %[t], %[t], -1\n\t" "s_min_u32 %[nx], %[nx], %[t]\n\t"
#define THEMIS_W_IS_LOWEST(K)                                                         \
  "s_bitcmp1_b32 %[ends], " #K "\n\t" "s_cbranch_scc0 .Lwn" #K "_%=\n\t"              \
  "s_and_b32 %[t], %[r" #K "], 0x1ff\n\t" "s_cmp_eq_u32 %[t], %[nx]\n\t"              \
  "s_cbranch_scc0 .Lwn" #K "_%=\n\t"                                                  \
  "s_mov_b32 %[rn], %[r" #K "]\n\t" "v_mov_b64_e32 %[f" #K "], %[nan]\n\t"            \
  "s_bitset0_b32 %[ends], " #K "\n\t" "s_bitset1_b32 %[idle], " #K "\n\t"             \
  "s_branch .Lwmd_%=\n\t" ".Lwn" #K "_%=:\n\t"
#define THEMIS_W_TAKE_TURN(K, P, LOG)                                                 \
  "s_bitcmp1_b32 %[idle], " #K "\n\t" "s_cbranch_scc0 .Lwa" #K "_%=\n\t"              \
  THEMIS_W_PICK_##P(K, a##K, ".Lwa" #K "_%=", LOG) ".Lwa" #K "_%=:\n\t"
#define THEMIS_W_SEVERAL(P, LOG)                                                      \
  ".Lwm_%=:\n\t" "s_mov_b32 %[nx], -1\n\t"                                            \
  THEMIS_W_LOWEST(0) THEMIS_W_LOWEST(1) THEMIS_W_LOWEST(2) THEMIS_W_LOWEST(3)         \
  THEMIS_W_IS_LOWEST(0) THEMIS_W_IS_LOWEST(1) THEMIS_W_IS_LOWEST(2) THEMIS_W_IS_LOWEST(3) \
  "s_branch .Lwend_%=\n\t"                                                            \
  ".Lwmd_%=:\n\t" "s_bitcmp1_b32 %[rn], 15\n\t" "s_cbranch_scc1 .Lwmn_%=\n\t"         \
  "s_and_b32 %[rc], %[rn], 0x7fff\n\t" "s_lshr_b32 %[t], %[rn], 22\n\t"               \
  "s_cmp_eq_u32 %[t], 0\n\t" "s_cbranch_scc1 .Lwm0_%=\n\t"                            \
  "s_cmp_eq_u32 %[t], 1\n\t" "s_cbranch_scc1 .Lwm1_%=\n\t"                            \
  "s_cmp_eq_u32 %[t], 2\n\t" "s_cbranch_scc1 .Lwm2_%=\n\t"                            \
  THEMIS_W_PUSH_##P(3, m3) "s_branch .Lwmn_%=\n\t"                                    \
  ".Lwm0_%=:\n\t" THEMIS_W_PUSH_##P(0, m0) "s_branch .Lwmn_%=\n\t"                    \
  ".Lwm1_%=:\n\t" THEMIS_W_PUSH_##P(1, m1) "s_branch .Lwmn_%=\n\t"                    \
  ".Lwm2_%=:\n\t" THEMIS_W_PUSH_##P(2, m2)                                            \
  ".Lwmn_%=:\n\t" "s_cmp_lg_u32 %[ends], 0\n\t" "s_cbranch_scc1 .Lwm_%=\n\t"          \
  ".Lwall_%=:\n\t" THEMIS_W_TAKE_TURN(0, P, LOG) THEMIS_W_TAKE_TURN(1, P, LOG)        \
  THEMIS_W_TAKE_TURN(2, P, LOG) THEMIS_W_TAKE_TURN(3, P, LOG) "s_branch .Lwnext_%=\n\t" \
  THEMIS_W_PUSH_AWAY_##P(0, m0) THEMIS_W_PUSH_AWAY_##P(1, m1)                         \
  THEMIS_W_PUSH_AWAY_##P(2, m2) THEMIS_W_PUSH_AWAY_##P(3, m3)                         \
  THEMIS_W_PICK_AWAY_##P(0, a0, ".Lwa0_%=", LOG) THEMIS_W_PICK_AWAY_##P(1, a1, ".Lwa1_%=", LOG) \
  THEMIS_W_PICK_AWAY_##P(2, a2, ".Lwa2_%=", LOG) THEMIS_W_PICK_AWAY_##P(3, a3, ".Lwa3_%=", LOG)

// The loop's place in the instruction stream (words behind a line of 64 bytes; us: the
// platforms of Table 2 0 135.3, 4 133.2, 6 136.7, 2 139.3; two first-in-first-out scenarios of 295
// chunks 0 and 4 424, 2 436, 6 438; as it came 135.4 and 438).
#define THEMIS_W_PLACE_FIFO1 ".p2align 6\n\t"
#define THEMIS_W_PLACE_FIFO2 ".p2align 6\n\t"
#define THEMIS_W_PLACE_SCF1 ".p2align 6\n\t.rept 4\n\ts_nop 0\n\t.endr\n\t"
#define THEMIS_W_PLACE_SCF2 ".p2align 6\n\t"
#define THEMIS_W_LOOP(P, LOG)                                                         \
  "s_nop 4\n\t" "s_branch .Lwall_%=\n\t" THEMIS_W_PLACE_##P                          \
  ".Lwnext_%=:\n\t"                                                                   \
  "v_min_f64 %[vt], %[f0], %[f1]\n\t" "v_min_f64 %[vn], %[f2], %[f3]\n\t"             \
  "v_min_f64 %[vt], %[vt], %[vn]\n\t"                                                 \
  "v_cmp_eq_f64_e64 vcc, %[f0], %[vt]\n\t" "v_cmp_eq_f64_e64 %[e1], %[f1], %[vt]\n\t" \
  "v_cmp_eq_f64_e64 %[e2], %[f2], %[vt]\n\t" "v_cmp_eq_f64_e64 %[e3], %[f3], %[vt]\n\t" \
  "s_and_b64 vcc, vcc, 1\n\t" "s_and_b64 %[e1], %[e1], 2\n\t" "s_or_b64 vcc, vcc, %[e1]\n\t" \
  "s_and_b64 %[e2], %[e2], 4\n\t" "s_and_b64 %[e3], %[e3], 8\n\t"                     \
  "s_or_b64 %[e2], %[e2], %[e3]\n\t" "s_or_b64 vcc, vcc, %[e2]\n\t"                   \
  "s_cbranch_scc0 .Lwend_%=\n\t" "v_mov_b64_e32 %[now], %[vt]\n\t"                   \
  "s_sub_u32 %[passes], %[passes], 1\n\t" "s_cbranch_scc1 .Lwend_%=\n\t"            \
  "s_mov_b32 %[ends], vcc_lo\n\t" "s_add_u32 %[t], vcc_lo, -1\n\t"                    \
  "s_and_b32 %[t], %[t], vcc_lo\n\t" "s_cbranch_scc1 .Lwm_%=\n\t"                     \
  "s_cmp_gt_u32 %[ends], 2\n\t" "s_cbranch_scc1 .Lw23_%=\n\t"                         \
  "s_bitcmp1_b32 %[ends], 1\n\t" "s_cbranch_scc1 .Lwc1_%=\n\t"                        \
  THEMIS_W_ENDED(0, 1, 2, 3, P, LOG) THEMIS_W_LINE THEMIS_W_ENDED(1, 0, 2, 3, P, LOG) \
  THEMIS_W_LINE ".Lw23_%=:\n\t" "s_bitcmp1_b32 %[ends], 3\n\t" "s_cbranch_scc1 .Lwc3_%=\n\t"        \
  THEMIS_W_ENDED(2, 0, 1, 3, P, LOG) THEMIS_W_LINE THEMIS_W_ENDED(3, 0, 1, 2, P, LOG) \
  THEMIS_W_SEVERAL(P, LOG)                                                            \
  ".Lwend_%=:\n\t" "s_mov_b64 exec, -1\n\t" "s_waitcnt lgkmcnt(0)\n\t" "s_nop 4\n\t"

#define THEMIS_W_DIM(K)                                                               \
  [f##K] "+&v"(d[K].finish), [z##K] "+&v"(d[K].busy), [h##K] "+&v"(d[K].head), [l##K] "+&v"(d[K].tail), \
  [q##K] "+&v"(d[K].queue), [g##K] "+&v"(d[K].log), [r##K] "+&s"(d[K].running), [x##K] "+&s"(d[K].lists), \
  [i##K] "+&s"(d[K].get), [o##K] "+&s"(d[K].put), [c##K] "+&s"(d[K].started)
#define THEMIS_W_TABLE(K)                                                             \
  [a##K] "v"(__double2loint(t.time[K])), [b##K] "v"(__double2hiint(t.time[K])), [n##K] "v"(t.next[K])

struct WaveResult {
  double t_done;
  double busy[kMaxDims];
  uint32_t executed[kMaxDims];
  bool ok;                    // false: some stage did not move the clock, or it overflowed
};

__device__ __forceinline__ uint32_t lds_offset(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

// kLog: the records each dimension executes go to lds.log.
// link: lane = chunk (only up to 64 chunks).
template <uint32_t kWords, bool kScf, bool kLog>
__device__ __forceinline__ WaveResult wave_events(const WaveTables& t, uint32_t stages, uint32_t C,
                                                  WaveDim (&d)[kMaxDims], uint32_t link,
                                                  WaveLds<kWords>& lds) {
  constexpr uint32_t kCap = 64u * kWords;
  double now = 0.0, vt, vn;
  uint32_t idle = 15u, rc, rn, nx, tmp, cls, ends, va, vd;
  uint64_t e1, e2, e3;
  const uint32_t log_bytes = 2u * kCap * (uint32_t)sizeof(uint16_t);
  // (the log is written once `started` has passed the 64 records)
  const uint32_t log_at = lds_offset(lds.log) + 2u * lane_id() - 128u;
  const uint32_t queue_at = lds_offset(lds.queue), link_at = lds_offset(lds.link);
  const uint32_t queue_lane = queue_at + 2u * lane_id();
  // every pass completes a stage; the two bounds end the loop, and keep the log
  // inside its block, whatever the records hold
  uint32_t passes = first_lane(stages * C);
  const uint32_t most = 2u * kCap;
#define THEMIS_W_RUN(P, LOG)                                                          \
  asm volatile(THEMIS_W_LOOP(P, LOG)                                                  \
      : THEMIS_W_DIM(0), THEMIS_W_DIM(1), THEMIS_W_DIM(2), THEMIS_W_DIM(3), [lk] "+&v"(link), \
        [now] "+&v"(now), [vt] "=&v"(vt), [vn] "=&v"(vn), [va] "=&v"(va), [vd] "=&v"(vd), [idle] "+&s"(idle), [passes] "+&s"(passes), \
        [rc] "=&s"(rc), [rn] "=&s"(rn), [nx] "=&s"(nx), [t] "=&s"(tmp), [c] "=&s"(cls), \
        [ends] "=&s"(ends), [e1] "=&s"(e1), [e2] "=&s"(e2), [e3] "=&s"(e3)            \
      : THEMIS_W_TABLE(0), THEMIS_W_TABLE(1), THEMIS_W_TABLE(2), THEMIS_W_TABLE(3),   \
        [nan] "v"(nan64()), [rb] "s"(log_bytes), [logat] "v"(log_at), [queueat] "s"(queue_at), \
        [queuelane] "v"(queue_lane), [linkat] "s"(link_at), [cap] "n"(kCap), [most] "s"(most) \
      : "vcc", "scc", "memory")
  if constexpr (kWords == 1u && kScf && kLog) THEMIS_W_RUN(SCF1, 1);
  else if constexpr (kWords == 1u && kScf) THEMIS_W_RUN(SCF1, 0);
  else if constexpr (kWords == 1u && kLog) THEMIS_W_RUN(FIFO1, 1);
  else if constexpr (kWords == 1u) THEMIS_W_RUN(FIFO1, 0);
  else if constexpr (kScf && kLog) THEMIS_W_RUN(SCF2, 1);
  else if constexpr (kScf) THEMIS_W_RUN(SCF2, 0);
  else if constexpr (kLog) THEMIS_W_RUN(FIFO2, 1);
  else THEMIS_W_RUN(FIFO2, 0);
#undef THEMIS_W_RUN

  WaveResult r;
  r.t_done = now;
  uint32_t started = 0u;
#pragma unroll
  for (uint32_t k = 0; k < (uint32_t)kMaxDims; ++k) {
    r.busy[k] = d[k].busy;
    r.executed[k] = d[k].started;
    started += d[k].started;
    // the records that did not fill the register
    const uint32_t full = d[k].started & ~63u;
    if (kLog && full + lane_id() < d[k].started) lds.log[k][(full + lane_id()) % (2u * kCap)] = (uint16_t)d[k].log;
  }
  // as in simulate_fast: every stage ran and completed, and none was too short
  // to move the clock
  r.ok = started == stages * C && idle == 15u && uniform(now < inf64() && now + 0.25 * t.t_min > now);
  return r;
}

// One single collective, all 64 lanes with the same arguments; code_at(c): order
// code of chunk c.  kLog: the records each dimension executes are left in lds.log.
enum class WaveOutcome { kMalformed, kDone, kNotTaken };   // (some order code; r holds the result; for wave_exact)
template <uint32_t kWords, bool kLog, typename CodeAt>
__device__ __forceinline__ WaveOutcome wave_simulate(const Scenario& s, double chunk, bool scf,
                                                     WaveLds<kWords>& lds, CodeAt code_at, WaveResult& r) {
  const uint32_t lane = lane_id();
  const uint32_t D = (uint32_t)s.D, C = s.C;
  const bool gather = s.ctype == THEMIS_COLL_ALL_GATHER;
  WaveDim d[kMaxDims];
#pragma unroll
  for (int k = 0; k < kMaxDims; ++k) {
    d[k].finish = nan64();
    d[k].busy = 0.0;
    d[k].running = d[k].started = d[k].get = d[k].put = 0u;
    d[k].lists = 0ull;
    d[k].head = d[k].tail = d[k].log = 0u;
  }
  // a6: every chunk waits at the dimension of its first stage, in chunk-id order
  uint32_t used = 0u;
  bool bad = false;
  for (uint32_t from = 0; from < C; from += 64u) {
    const uint32_t c = from + lane;
    const bool exists = c < C;
    const uint32_t given = exists ? code_at(c) : 0u;
    bad = bad || (exists && !order_code_ok(given, s.D));
    const uint32_t code = gather ? reverse_code(given, s.D) : given;
    const uint32_t rank = ring_order_rank(code, D) % kWaveOrders;
    const uint32_t k0 = (code >> (gather ? 2u * (D - 1u) : 0u)) & 3u;
    used |= exists ? 1u << rank : 0u;
    const uint32_t rec = c | (rank + (gather ? kWaveOrders : 0u)) << kWaveStateShift;
#pragma unroll
    for (uint32_t k = 0; k < (uint32_t)kMaxDims; ++k) {
      const bool here = exists && k0 == k;
      const uint64_t m = __builtin_amdgcn_ballot_w64(here);
      const uint32_t at = d[k].put + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                         __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
      if (here) lds.queue[k][at] = (uint16_t)rec;
      d[k].put += (uint32_t)__builtin_popcountll(m);
    }
  }
  for (int off = 32; off > 0; off >>= 1) used |= (uint32_t)__shfl_xor((int)used, off);
  used = first_lane(used);
  if (uniform(bad)) return WaveOutcome::kMalformed;
  __syncthreads();
  uint32_t link = 0u;
  if (gather && scf) {
    // the size of the first wait is the smallest there is: these chunks
    // are on lists from the start
#pragma unroll
    for (uint32_t k = 0; k < (uint32_t)kMaxDims; ++k) {
      for (uint32_t p = lane; p + 1u < d[k].put; p += 64u)
        lds.link[lds.queue[k][p] & kWaveIdMask] = lds.queue[k][p + 1u];
      if (d[k].put != 0u) {
        d[k].lists = 1ull;
        d[k].head = lds.queue[k][0];
        d[k].tail = lds.queue[k][d[k].put - 1u];
      }
      d[k].get = d[k].put;
    }
    __syncthreads();
    if (kWords == 1u) link = lds.link[lane];
  }
#pragma unroll
  for (uint32_t k = 0; k < (uint32_t)kMaxDims; ++k) {
    d[k].queue = lds.queue[k][lane];
    d[k].put = first_lane(d[k].put);
    d[k].get = first_lane(d[k].get);
    d[k].lists = first_lane((uint32_t)d[k].lists);   // (class 0 at most)
  }
  WaveTables t;
  wave_tables(s, chunk, scf, used, t, true);
  if (!t.normal) return WaveOutcome::kNotTaken;
  const uint32_t stages = s.ctype == THEMIS_COLL_ALL_REDUCE ? 2u * D : D;
  r = scf ? wave_events<kWords, true, kLog>(t, stages, C, d, link, lds)
          : wave_events<kWords, false, kLog>(t, stages, C, d, link, lds);
  __syncthreads();
  return r.ok ? WaveOutcome::kDone : WaveOutcome::kNotTaken;
}

// What the event loop does not take (a stage that does not move the clock,
// sizes outside the normal range, overflow), one wavefront per evaluation, by
// the definition itself: every pass looks at all chunks, their sizes and
// arrival times (see simulate_generic, whose passes these are).
template <uint32_t kWords>
struct WaveExactLds {
  double arrival[64u * kWords], size[64u * kWords];
  uint16_t meta[64u * kWords];   // stage (bits 0-3) | running (bit 4) | order code (bits 8-15)
};

template <uint32_t kWords, typename CodeAt, typename Put>
__device__ __forceinline__ WaveResult wave_exact(const Scenario& s, double chunk, bool scf,
                                                 WaveExactLds<kWords>& m, CodeAt code_at, Put put) {
  const int D = s.D;
  const uint32_t C = s.C;
  const bool gather = s.ctype == THEMIS_COLL_ALL_GATHER;
  const int last_stage = s.ctype == THEMIS_COLL_ALL_REDUCE ? 2 * D : D;
  for (uint32_t c = lane_id(); c < C; c += 64u) {
    m.arrival[c] = 0.0;
    m.size[c] = chunk;
    m.meta[c] = (uint16_t)(code_at(c) << 8);
  }
  __syncthreads();
  int serving[kMaxDims] = {-1, -1, -1, -1};
  double finish[kMaxDims] = {0.0, 0.0, 0.0, 0.0};
  WaveResult r;
#pragma unroll
  for (int k = 0; k < kMaxDims; ++k) { r.busy[k] = 0.0; r.executed[k] = 0u; }
  double now = 0.0, last_done = 0.0;
  for (uint32_t pass = 0; pass < 2u * (uint32_t)D * C + 8u; ++pass) {
#pragma unroll
    for (int k = 0; k < kMaxDims; ++k) {
      if (k >= D || serving[k] >= 0) continue;
      uint32_t best = ~0u;
      double bsize = inf64(), barr = inf64();
      for (uint32_t c = lane_id(); c < C; c += 64u) {
        const uint32_t w = m.meta[c];
        const int stage = (int)(w & 15u);
        if (stage >= last_stage || (w & kMetaRunning)) continue;
        const int pos = stage < D ? stage : 2 * D - 1 - stage;
        if ((int)((w >> (8 + 2 * pos)) & 3u) != k) continue;
        const double sz = scf ? m.size[c] : 0.0, arr = m.arrival[c];
        if (best == ~0u || sz < bsize || (sz == bsize && arr < barr)) { best = c; bsize = sz; barr = arr; }
      }
      for (int off = 32; off > 0; off >>= 1) {
        const uint32_t oc = (uint32_t)__shfl_xor((int)best, off);
        const double os = __shfl_xor(bsize, off), oa = __shfl_xor(barr, off);
        const bool other = oc != ~0u && (best == ~0u || os < bsize ||
                                         (os == bsize && (oa < barr || (oa == barr && oc < best))));
        if (other) { best = oc; bsize = os; barr = oa; }
      }
      best = first_lane(best);
      if (best == ~0u) continue;
      const uint32_t w = m.meta[best];
      const int stage = (int)(w & 15u);
      double x = m.size[best];
      if (gather) {
        x = x * (double)s.P[k];
      } else if (stage >= D) {
        x = chunk;
        for (int j = 0; j < 2 * D - 1 - stage; ++j)
          x = x / (double)sel4((int)((w >> (8 + 2 * j)) & 3u), s.P[0], s.P[1], s.P[2], s.P[3]);
      }
      double time = x * s.coef[k];
      if (s.has_fix) time = s.fix[k] + time;
      finish[k] = now + time;
      r.busy[k] = r.busy[k] + time;
      serving[k] = (int)best;
      __syncthreads();
      if (lane_id() == 0u) m.meta[best] = (uint16_t)(w | kMetaRunning);
      __syncthreads();
      put((uint32_t)k, r.executed[k], (best << 1) | ((gather || stage >= D) ? 1u : 0u));
      r.executed[k]++;
    }
    double next = inf64();
#pragma unroll
    for (int k = 0; k < kMaxDims; ++k)
      if (serving[k] >= 0 && finish[k] < next) next = finish[k];
    if (!uniform(next < inf64())) break;
    now = next;
#pragma unroll
    for (int k = 0; k < kMaxDims; ++k) {
      if (serving[k] >= 0 && uniform(finish[k] == now)) {
        const uint32_t c = (uint32_t)serving[k];
        const uint32_t w = m.meta[c];
        const int stage = (int)(w & 15u);
        const double pk = (double)s.P[k];
        const double size = m.size[c];
        __syncthreads();
        if (lane_id() == 0u) {
          m.size[c] = (!gather && stage < D) ? size / pk : size * pk;
          m.arrival[c] = now;
          m.meta[c] = (uint16_t)((w & ~(15u | kMetaRunning)) | (uint32_t)(stage + 1));
        }
        __syncthreads();
        serving[k] = -1;
        if (stage + 1 == last_stage) last_done = now;
      }
    }
  }
  r.t_done = last_done;
  bool finite = last_done < inf64();
#pragma unroll
  for (int k = 0; k < kMaxDims; ++k) finite = finite && r.busy[k] < inf64();
  r.ok = finite;
  return r;
}

}  // namespace themis
