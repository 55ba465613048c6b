// Event loop with four lanes per evaluation: lane j of a quad owns dimension j
// of the network (its FIFO lists per size class, the stage it serves, its
// finish and busy time), the four share one LDS block, and the clock of the
// evaluation is the minimum of the quad's finish times (paper Sec. 4.3 for the
// queues, Sec. 4.6.2 for the simulation that keeps every NPU's view the same).
//
// The mapping with one lane per evaluation keeps a whole evaluation's records
// in that lane's LDS block; at 512 chunks that is 80 KiB per wavefront and two
// wavefronts per CU, each alone on its SIMD and waiting out every dependent
// instruction and every LDS read (30,001 scenarios of 200 chunks, 8 thresholds x 2
// policies: 10.5 ms, here 4.5).  Here a wavefront holds 16 evaluations in
// 20 KiB, eight wavefronts fit a CU, and a lane never has to pick one of four
// dimensions' registers.
//
// A pass of the loop delivers one completion per evaluation: the quad agrees on
// the chunk (the lowest id among the stages that end now), the lane that owns
// the dimension it waits for next appends it to its list, and every idle lane
// with chunks waiting starts one.  All that a lane reads or writes in LDS is its
// own dimension's, so nothing has to be ordered between lanes, and a pass is two
// dependent LDS trips: the ends of the list served (and of the one appended to),
// then the link behind its first chunk together with what the stage does.
// (Before, with the lane whose stage ends appending, one loop round per completion
// and the stage derived from the order field: 133 vector instructions a pass, now
// some 65; 512-chunk sweep of 65,536 networks, 8 thresholds x 2 policies, 47.3 ->
// 29.7 ms.  A wavefront alone on its SIMD takes 860 clocks a pass, four on one 350
// each: the first is the chain of dependent instructions and the two trips, the
// second issue.  The link behind a chunk that starts is stored whether the list goes on or
// not, with no branch around it: 20,001 scenarios of 250 chunks 1,013 -> 890 us.)
// Wavefronts of first-in-first-out evaluations alone have a loop without lists in LDS
// (quad_loop_fifo).
//
// A record names a chunk and its state: bits 0-8 the chunk, 9-13 its order's
// place among those of D dimensions, 14 the phase (up to three dimensions the
// phase may follow the order in bit 12).  Lists hold records, a link
// the record of the next chunk, so nothing else is kept per chunk.
//
// Per evaluation (quad g of the wavefront): first | last << 16 of list q = kClasses *
// dimension + class at byte 64 * q + 4 * g; behind the lists the link of chunk c, 16
// bits, at byte 32 * c + 2 * g.  (One shift and add; the quads' words of one index are
// in different banks.  A dimension where nothing waits reads a list behind its own
// without a use for it: one of the next dimension, or links.)
#pragma once

#include "themis_fast.hpp"
#include "themis_ring.hpp"

namespace themis {

template <uint32_t kChunks, uint32_t kClasses, uint32_t kOrderBits = 5>
struct LayoutQuad {
  static constexpr uint32_t kCap = kChunks, kPerDim = kClasses;
  static constexpr uint32_t kPhaseBit = 9u + kOrderBits;   // of a record
  static constexpr uint32_t kQuads = (uint32_t)kBlock / 4u;
  static constexpr uint32_t kLinksAt = 64u * 4u * kClasses;
  static constexpr uint32_t kBytes = kLinksAt + 32u * kChunks;
  static constexpr uint32_t kIdMask = 0x1ffu;
  static constexpr uint32_t kWavesPerSimd = kChunks <= 128u ? 4u : 2u;
  // (a list's ends are written as a word and, where a chunk leaves, as its lower half, and
  // what makes a scenario's tables has used the place for sizes)
  typedef uint16_t __attribute__((may_alias)) Half;
  typedef uint32_t __attribute__((may_alias)) Word;
  // link of the chunk of record rec (the shifts end in an address: one instruction each)
  static __device__ __forceinline__ Half* link(uint8_t* block, uint32_t rec) {
    return (Half*)(block + kLinksAt + (((rec << 5) & (kIdMask << 5)) | ((threadIdx.x >> 2) * 2u)));
  }
  // ends of the lane's list of a class
  static __device__ __forceinline__ Word* ends(uint8_t* block, uint32_t cls) {
    return (Word*)(block + (threadIdx.x >> 2) * 4u + 64u * kPerDim * (threadIdx.x & 3u) + (cls << 6));
  }
};

// Values of the quad's other lanes: quad_perm [1,0,3,2] and [2,3,0,1].
__device__ __forceinline__ uint32_t quad_swap1(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xb1, 0xf, 0xf, true);
}
__device__ __forceinline__ uint32_t quad_swap2(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4e, 0xf, 0xf, true);
}
// Value of the quad's lane j.
template <int j>
__device__ __forceinline__ uint32_t quad_lane(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x55 * j, 0xf, 0xf, true);
}
__device__ __forceinline__ uint32_t quad_min_u32(uint32_t v) {
  v = min(v, quad_swap1(v));
  return min(v, quad_swap2(v));
}
__device__ __forceinline__ uint32_t quad_or(uint32_t v) {
  v |= quad_swap1(v);
  return v | quad_swap2(v);
}
__device__ __forceinline__ uint32_t quad_sum(uint32_t v) {
  v += quad_swap1(v);
  return v + quad_swap2(v);
}
// Minimum of the quad's doubles, quiet NaNs skipped (NaN if all four are).
__device__ __forceinline__ double quad_min_f64(double v) {
  double o = __hiloint2double((int)quad_swap1((uint32_t)__double2hiint(v)),
                              (int)quad_swap1((uint32_t)__double2loint(v)));
  v = min_f64(v, o);
  o = __hiloint2double((int)quad_swap2((uint32_t)__double2hiint(v)),
                       (int)quad_swap2((uint32_t)__double2loint(v)));
  return min_f64(v, o);
}
// The double of the quad's lane k ^ j.
__device__ __forceinline__ double quad_other(double v, uint32_t j) {
  const uint32_t hi = (uint32_t)__double2hiint(v), lo = (uint32_t)__double2loint(v);
  const auto swap3 = [](uint32_t x) { return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x1b, 0xf, 0xf, true); };
  return j == 1u ? __hiloint2double((int)quad_swap1(hi), (int)quad_swap1(lo))
       : j == 2u ? __hiloint2double((int)quad_swap2(hi), (int)quad_swap2(lo))
                 : __hiloint2double((int)swap3(hi), (int)swap3(lo));
}
// The double of the one lane of the quad that says so.
__device__ __forceinline__ double quad_pick(double v, bool mine) {
  return __hiloint2double((int)quad_or(mine ? (uint32_t)__double2hiint(v) : 0u),
                          (int)quad_or(mine ? (uint32_t)__double2loint(v) : 0u));
}
// Largest value of the wavefront.
__device__ __forceinline__ uint32_t quad_wave_max(uint32_t v) {
  for (int off = 32; off > 0; off >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, off));
  return v;
}
// Place of an order code among the orders of D dimensions (lexicographic).
__device__ __forceinline__ uint32_t quad_order(uint32_t code, uint32_t D) {
  const uint32_t r = ring_order_rank(code, D);
  return D >= 4u ? r : D == 3u ? r / 6u * 2u + r % 6u / 2u : r / 6u;
}

// What the stage of a chunk on dimension k does, as far as it does not depend on
// the sizes: by row + 32 * phase, k (quad_stage_at); the rows of the orders of D
// dimensions start at quad_row(D), where those of four leave room (an order of one
// dimension has the third column of one of two).  Bits 1-3 the dimension the chunk waits for
// next (4: it is finished), 9-14 its row and phase then, 17-22 four times the mask
// of its reduced dimensions then; bits 0, 8, 16, 24: dimension 0, 1, 2, 3 comes
// before k in its order.
// The second half is the same where a chunk's last Reduce-Scatter and its first All-Gather, on the
// same dimension, are one stage (bit 31) that takes the time of one twice.  Under
// Smallest-Chunk-First nothing comes between them: the chunk is smaller then than any that
// waits there, and moves the same bytes again.
// (One array for both, since they are copied to LDS in one go.)
constexpr uint32_t kQuadStageWords = 64u * 4u;   // of each half
struct QuadStages {
  uint32_t v[2u * kQuadStageWords];
  uint8_t code[4][24];   // the order codes themselves, by (dimensions - 1)
};
__host__ __device__ constexpr uint32_t quad_stage_at(uint32_t row, uint32_t column) { return 4u * row + column; }
// Word i of the two halves, as the copies read it.
__host__ __device__ constexpr uint32_t quad_stage_word(const QuadStages& t, uint32_t i) { return t.v[i]; }
__host__ __device__ constexpr uint32_t quad_row(uint32_t D) { return D >= 4u ? 0u : D == 3u ? 24u : 30u; }
__host__ __device__ constexpr uint32_t quad_column(uint32_t D) { return D == 1u ? 2u : 0u; }
constexpr QuadStages quad_stages() {
  QuadStages t{};
  for (uint32_t D = 1; D <= 4; ++D) {
    uint32_t perm[4] = {0, 1, 2, 3}, n = 0;
    const uint32_t full = (1u << D) - 1u;
    for (uint32_t i = 0; i < 256u; ++i) {   // field j of i, last field fastest: lexicographic
      bool ok = true;
      uint32_t seen = 0;
      for (uint32_t j = 0; j < 4u; ++j) {
        perm[j] = (i >> (2u * (3u - j))) & 3u;
        if (j < D ? perm[j] >= D || ((seen >> perm[j]) & 1u) != 0u : perm[j] != 0u) ok = false;
        if (j < D) seen |= 1u << perm[j];
      }
      if (!ok) continue;
      uint32_t before = 0;
      const uint32_t row = quad_row(D) + n;
      t.code[D - 1u][n] = 0;
      for (uint32_t j = 0; j < D; ++j) {
        t.code[D - 1u][n] = (uint8_t)(t.code[D - 1u][n] | perm[j] << (2u * j));
        const uint32_t k = perm[j], with = before | (1u << k), column = k + quad_column(D);
        const bool last = with == full;
        uint32_t bits = 0;
        for (uint32_t d = 0; d < 4u; ++d) bits |= ((before >> d) & 1u) << (8u * d);
        t.v[quad_stage_at(row, column)] = (last ? k : perm[j + 1u < 4u ? j + 1u : 3u]) << 1 | (row + (last ? 32u : 0u)) << 9 |
                                          (4u * with) << 17 | bits;
        t.v[quad_stage_at(32u + row, column)] =
            (j == 0u ? 4u : perm[j - (j ? 1u : 0u)]) << 1 | (row + 32u) << 9 | (4u * before) << 17 | bits;
        before = with;
      }
      for (uint32_t k = 0; k < D; ++k) {
        const uint32_t scatter = quad_stage_at(row, k + quad_column(D)), gather = quad_stage_at(32u + row, k + quad_column(D));
        t.v[kQuadStageWords + scatter] = ((t.v[scatter] >> 14) & 1u) != 0u ? t.v[gather] | 1u << 31 : t.v[scatter];
        t.v[kQuadStageWords + gather] = t.v[gather];
      }
      ++n;
    }
  }
  return t;
}
__device__ const QuadStages g_quad_stages = quad_stages();

// Stages of a chunk on the lane's dimension where the NPU counts are powers of
// two (records hold quad_row() + order).  A stage takes 2^-e times as long as on the
// whole chunk, e the sum of log2 P over the dimensions before: the product with the
// power of two may come after the one with the latency as long as no result leaves
// the normal range (t_min).
// A running stage, as the quad passes it on: bits 1-3 the dimension the chunk waits
// for then (4: none), 9-14 its row and phase then, 16-19 the list it joins, 23-31 the
// chunk.
// The stage tables are in LDS behind the lists (2 KiB, 60 clocks nearer than the
// caches) where that costs no wavefront: up to 256 chunks; the one without turns in the
// place of the lists' ends where the wavefront does without them (fifo).
template <typename L, bool kFix>
struct QuadPow2 {
  static constexpr bool kTableInLds = L::kCap <= 256u;
  static constexpr uint32_t kTableAt = kTableInLds ? L::kBytes : 0u;
  static constexpr uint32_t kTable = 4u * kQuadStageWords;   // bytes of each
  static constexpr uint32_t kBytes = L::kBytes + (kTableInLds ? 2u * kTable : 0u);
  static_assert(kTableInLds || L::kLinksAt >= kTable, "a table fits the place of the lists' ends");
  static constexpr double kShortest = 2.2250738585072014e-308;   // (see above)
  static constexpr uint32_t kNobody = ~0u;   // above all stages, for dimension 7, list 31 (a place behind the lists)
  double whole, fix;
  uint64_t ranktab;
  int less;         // -log2 P_k in byte k
  uint8_t* block;
  uint32_t at, wanted;
  bool fifo;        // no evaluation of the wavefront has more than one class
  __device__ __forceinline__ QuadPow2(const Scenario& s, const Pow2Model& m, uint32_t k, void* lds)
      : whole(m.fs.base * sel4((int)k, s.coef[0], s.coef[1], s.coef[2], s.coef[3])),
        fix(kFix ? sel4((int)k, s.fix[0], s.fix[1], s.fix[2], s.fix[3]) : 0.0), ranktab(m.ranktab), less(0),
        block((uint8_t*)lds),
        at(4u * ((k + quad_column((uint32_t)s.D)) & 3u) | (m.ranktab != 0ull && !m.rs_only() ? kTable : 0u)),
        // a stand-alone Reduce-Scatter is finished where the phase would turn
        wanted(m.rs_only() ? 14u | 0x4000u : 14u), fifo(__builtin_amdgcn_ballot_w64(m.ranktab != 0ull) == 0ull) {
#pragma unroll
    for (uint32_t d = 0; d < 4u; ++d) less |= (int)((0u - (m.fs.epack >> (8u * d) & 0xffu) & 0xffu) << (8u * d));
    if (kTableInLds || fifo)
      for (uint32_t j = 0; j < (kTableInLds ? 8u : 4u); ++j)
        ((typename L::Word*)(block + kTableAt))[64u * j + threadIdx.x % 64u] = quad_stage_word(g_quad_stages, 64u * j + threadIdx.x % 64u);
    __syncthreads();
  }
  __device__ __forceinline__ bool goes_to(uint32_t given, uint32_t k) const { return (given & wanted) == 2u * k; }
  static __device__ __forceinline__ uint32_t list(uint32_t given) { return (given >> 16) & 31u; }
  static __device__ __forceinline__ uint32_t record(uint32_t given) { return (given & 0x7e00u) | given >> 23; }
  // rec: the chunk's record in the low half; kFifo: on a wavefront of one class; turned: it takes
  // the time twice
  template <bool kFifo>
  __device__ __forceinline__ uint32_t stage(uint32_t rec, double& time, bool& turned) const {
    const uint8_t* const table = kTableInLds || kFifo ? block + kTableAt : (const uint8_t*)g_quad_stages.v;
    const uint32_t v = *(const typename L::Word*)(table + (((rec >> 5) & 0x3f0u) | at));
    time = ldexp(whole, __builtin_amdgcn_sdot4((int)(v & 0x01010101u), less, 0, true));
    if (kFix) time = fix + time;
    turned = (int)v < 0;
    if (kFifo) return (v & 0x7e0eu) | rec << 23;
    const uint32_t cls = (uint32_t)(ranktab >> ((v >> 17) & 63u)) & 15u;
    return ((v & 0x7e0eu) | rec << 23) | cls << 16;
  }
};

// Stages on the lane's dimension from tables of the evaluation itself, whatever
// its NPU counts are: a division by an arbitrary count rounds, so a chunk's sizes
// and times depend on its whole order, and are made by the model's own sequence
// of divisions and multiplications, once per order that some chunk has.
// In LDS behind the lists (quad g): time of order o on dimension k, binary64, at
// 128 * (4 * o + k) + 8 * g, and what the completion does, 16 bits (0-2 the dimension
// the chunk waits for then, 3-8 the list it joins, 9-14 its state, 15: turned, see QuadStages), at
// 32 * (4 * state + k) + 2 * g (state: order and phase as in a record); a running
// stage is these bits and the chunk from bit 23 on; size classes of (state, k) while these are made, 8 bits, at
// 16 * (4 * state + k) + g.
// L: layout; kDims: up to three dimensions (six orders, at most twelve sizes that
// wait for one dimension), or four (24, 48).
template <typename L, uint32_t kDims>
struct QuadTable {
  static constexpr uint32_t kOrders = kDims == 4u ? 24u : 6u;
  static constexpr uint32_t kStates = (L::kPhaseBit == 14u ? 32u : 8u) + kOrders;
  static constexpr uint32_t kTimes = L::kBytes, kDoes = kTimes + 512u * kOrders;
  // (the classes' place is the links', where it is large enough)
  static constexpr bool kInLinks = 64u * kStates <= 32u * L::kCap;
  static constexpr uint32_t kClassesAt = kInLinks ? L::kLinksAt : kDoes + 128u * kStates;
  static constexpr uint32_t kBytes = kDoes + 128u * kStates + (kInLinks ? 0u : 64u * kStates);
  static_assert(64u * 4u * L::kPerDim >= 512u * kOrders, "the sizes of one phase fit the place of the lists");
  static constexpr double kShortest = 0.0;   // times may leave the normal range
  static constexpr uint32_t kNobody = 0xffff0004u;   // above all stages, for dimension 4, list 0
  uint8_t* block;
  double t_min;
  uint32_t cls0;
  bool fifo;        // as in QuadPow2
  static __device__ __forceinline__ uint32_t quad8() { return (threadIdx.x >> 2) * 8u; }
  static __device__ __forceinline__ double* f64_at(uint8_t* b, uint32_t o, uint32_t k) {
    return (double*)(b + (o << 9 | k << 7 | quad8()));
  }
  static __device__ __forceinline__ uint16_t* does_at(uint8_t* b, uint32_t state, uint32_t k) {
    return (uint16_t*)(b + kDoes + (state << 7 | k << 5 | (threadIdx.x >> 2) * 2u));
  }
  static __device__ __forceinline__ uint8_t* class_at(uint8_t* b, uint32_t state, uint32_t k) {
    return b + kClassesAt + (state << 6 | k << 4 | threadIdx.x >> 2);
  }
  static __device__ __forceinline__ uint32_t state_of(uint32_t order, uint32_t phase) {
    return order | phase << (L::kPhaseBit - 9u);
  }
  // used: bit o says that some chunk has order o.  All lanes of the wavefront.
  __device__ __forceinline__ QuadTable(const Scenario& s, double chunk, bool scf, uint32_t used, void* lds)
      : block((uint8_t*)lds), t_min(inf64()), cls0(0u),
        fifo(__builtin_amdgcn_ballot_w64(scf) == 0ull) {
    const uint32_t k = threadIdx.x & 3u, D = min((uint32_t)s.D, kDims);
    const bool gather = s.ctype == THEMIS_COLL_ALL_GATHER, rs_only = s.ctype == THEMIS_COLL_REDUCE_SCATTER;
    uint8_t* const rs = block + kTimes;        // sizes before the Reduce-Scatter stages, then the times
    uint8_t* const ag = block;                 // sizes before the All-Gather stages, in the place of the lists
    // sizes: lane j of the quad takes the orders j, j + 4, ..  (NaN, below no
    // size, where there is none)
    constexpr uint32_t kTakes = (kOrders + 3u) / 4u;
    uint32_t codes[kTakes];
#pragma unroll
    for (uint32_t j = 0; j < kTakes; ++j) codes[j] = g_quad_stages.code[(D - 1u) & 3u][min(k + 4u * j, kOrders - 1u)];
    double least = inf64();
#pragma unroll
    for (uint32_t j4 = 0; j4 < kTakes; ++j4) {
      const uint32_t o = k + 4u * j4;
      if (o >= kOrders) break;
      const bool has = ((used >> o) & 1u) != 0u;
      const uint32_t code = has ? codes[j4] : 0xe4u;
      double x = has ? chunk : nan64();
      for (uint32_t j = 0; j < kDims; ++j) {
        const uint32_t kj = j < D ? (code >> (2u * j)) & 3u : j;
        *f64_at(rs, o, kj) = j < D && !gather ? x : nan64();
        if (!gather && j < D) x = x / (double)sel4((int)kj, s.P[0], s.P[1], s.P[2], s.P[3]);
      }
      least = min_f64(least, x);
      for (uint32_t j = kDims; j-- > 0u;) {
        const uint32_t kj = j < D ? (code >> (2u * j)) & 3u : j;
        *f64_at(ag, o, kj) = j < D && !rs_only ? x : nan64();
        if (j < D) x = x * (double)sel4((int)kj, s.P[0], s.P[1], s.P[2], s.P[3]);
      }
    }
    __syncthreads();
    // Classes: the number of smaller sizes among those that wait for the lane's dimension.
    // The lane's own sizes and counts are in registers, and each size is read once for all
    // of them (each comparison with a read of its own: 57 us of 264 for 750 turns of four
    // dimensions, 64 chunks), on four dimensions those of orders that some chunk has, since a
    // few chunks have few (all of them: 8,000 scenarios of 2 chunks 52 us for 36, 65,536 of
    // 4 chunks 238 for 182, of 16 378 for 346).  A chunk waits for its first stage at its whole size.
    if (scf) {
      uint32_t rank[2u * kOrders];
      double own[2u * kOrders];
#pragma unroll
      for (uint32_t i = 0; i < 2u * kOrders; ++i) {
        rank[i] = 0u;
        own[i] = *f64_at(i < kOrders ? rs : ag, i % kOrders, k);
      }
      auto count = [&](uint32_t o) {
        const double v = *f64_at(rs, o, k), w = *f64_at(ag, o, k);
        cls0 += (v < chunk ? 1u : 0u) + (w < chunk ? 1u : 0u);
#pragma unroll
        for (uint32_t i = 0; i < 2u * kOrders; ++i) rank[i] += (v < own[i] ? 1u : 0u) + (w < own[i] ? 1u : 0u);
      };
      if (kDims < 4u)   // (six orders: no faster by the ones in use)
        for (uint32_t o = 0; o < kOrders; ++o) count(o);
      else
        for (uint32_t m = used; m != 0u; m &= m - 1u) count((uint32_t)__builtin_ctz(m));
#pragma unroll
      for (uint32_t i = 0; i < 2u * kOrders; ++i) *class_at(block, state_of(i % kOrders, i / kOrders), k) = (uint8_t)rank[i];
    }
    __syncthreads();
    const double coef = sel4((int)k, s.coef[0], s.coef[1], s.coef[2], s.coef[3]);
    const double fix = sel4((int)k, s.fix[0], s.fix[1], s.fix[2], s.fix[3]);
    // (sizes that have left the normal range may be equal)
    least = quad_min_f64(least);
    const bool turns = scf && !rs_only && least >= 2.2250738585072014e-308;
    const double grow = gather ? (double)sel4((int)k, s.P[0], s.P[1], s.P[2], s.P[3]) : 1.0;
    const uint32_t* const stages = g_quad_stages.v + (turns ? kQuadStageWords : 0u) +
                                   quad_stage_at(quad_row(D), (k + quad_column(D)) & 3u);
    constexpr uint32_t kAtOnce = kOrders % 4u == 0u ? 4u : 3u;   // (loads that do not wait for each other)
    for (uint32_t from = 0; from < kOrders; from += kAtOnce) {
      uint32_t given[2][kAtOnce];
#pragma unroll
      for (uint32_t j = 0; j < kAtOnce; ++j) {
        given[0][j] = stages[4u * min(from + j, 31u - quad_row(D))];
        given[1][j] = stages[4u * (32u + min(from + j, 31u - quad_row(D)))];
      }
#pragma unroll
      for (uint32_t j = 0; j < kAtOnce; ++j) {
        const uint32_t o = from + j;
        if (k >= D || ((used >> o) & 1u) == 0u) continue;
        const double moved = gather ? *f64_at(ag, o, k) * grow : *f64_at(rs, o, k);
        double time = moved * coef;
        if (s.has_fix) time = fix + time;
        *f64_at(rs, o, k) = time;
        t_min = min_f64(t_min, time);
#pragma unroll
        for (uint32_t phase = 0; phase < 2u; ++phase) {
          if (phase == 0u ? gather : rs_only) continue;
          const uint32_t v = given[phase][j];
          const uint32_t turned = (v >> 14) & 1u, next = state_of(o, turned);
          const uint32_t to = rs_only && turned != 0u ? 4u : (v >> 1) & 7u;
          const uint32_t cls = scf && to < 4u ? *class_at(block, next, to) : 0u;
          *does_at(block, state_of(o, phase), k) = (uint16_t)(to | cls << 3 | next << 9 | (v >> 31) << 15);
        }
      }
    }
    t_min = quad_min_f64(t_min);
    __syncthreads();
  }
  static __device__ __forceinline__ bool goes_to(uint32_t given, uint32_t k) { return (given & 7u) == k; }
  static __device__ __forceinline__ uint32_t list(uint32_t given) { return (given >> 3) & 63u; }
  static __device__ __forceinline__ uint32_t record(uint32_t given) { return (given & 0x7e00u) | given >> 23; }
  template <bool kFifo>
  __device__ __forceinline__ uint32_t stage(uint32_t rec, double& time, bool& turned) const {
    const uint32_t k = threadIdx.x & 3u;
    time = *(const double*)(block + kTimes + ((rec & (L::kPhaseBit == 14u ? 0x3e00u : 0xe00u)) | (k << 7 | quad8())));
    const uint32_t v = *(const uint16_t*)(block + kDoes + (((rec >> 2) & (L::kPhaseBit == 14u ? 0x1f80u : 0x780u)) |
                                                           (k << 5 | (threadIdx.x >> 2) * 2u)));
    turned = (v & 0x8000u) != 0u;
    return v | rec << 23;
  }
};

// Alg. 1 with four lanes per collective, NPU counts that are not powers of two:
// lane k keeps dimension k's load, its place in the order is the number of loads
// below it, and it divides the chunk by the counts of the dimensions before it.
// All lanes of the wavefront; chunks: 0 where there is nothing to plan.
// kExact: IEEE divisions, for sizes that leave the normal range.
// emit(c, code): the same in the four lanes.  load: of the lane's dimension.
template <bool kExact, typename Emit>
__device__ __forceinline__ void plan_quad(const Scenario& s, double chunk, bool themis, bool rel, double thr,
                                          uint32_t chunks, double& load, Emit emit) {
  const uint32_t k = threadIdx.x & 3u, D = (uint32_t)s.D;
  const bool used = k < D, gather = s.ctype == THEMIS_COLL_ALL_GATHER, twice = s.ctype == THEMIS_COLL_ALL_REDUCE;
  const double coef = sel4((int)k, s.coef[0], s.coef[1], s.coef[2], s.coef[3]);
  const double mine = (double)sel4((int)k, s.P[0], s.P[1], s.P[2], s.P[3]);
  double inverse[kMaxDims];
#pragma unroll
  for (int d = 0; d < kMaxDims; ++d) inverse[d] = 1.0 / (double)s.P[d];
  // the threshold where this dimension is the least loaded
  const double below = rel ? thr * ((gather ? chunk * mine : chunk) * coef) : thr;
  const double fix = sel4((int)k, s.fix[0], s.fix[1], s.fix[2], s.fix[3]);
  load = used ? (twice ? fix + fix : fix) : inf64();
  const uint32_t most = (uint32_t)__builtin_amdgcn_readfirstlane((int)quad_wave_max(chunks));
  for (uint32_t c = 0; c < most; ++c) {
    uint32_t before = 0u;   // the dimensions before this one in the stable ascending order
#pragma unroll
    for (uint32_t j = 1; j < 4u; ++j) {
      const uint32_t other = k ^ j;
      const double l = quad_other(load, j);
      before += l < load || (l == load && other < k) ? 1u : 0u;
    }
    const double lo = quad_min_f64(load), hi = -quad_min_f64(used ? -load : inf64());
    const double at_least = quad_pick(below, before == 0u);
    const bool sorted = themis && !(hi - lo < at_least);
    const uint32_t rank = sorted ? before : k;
    const uint32_t place = gather ? D - 1u - rank : rank;
    const uint32_t code = quad_or(used ? k << (2u * place) : 0u);
    double x = chunk;
#pragma unroll
    for (uint32_t j = 0; j < 3u; ++j) {
      const int d = (int)((code >> (2u * j)) & 3u);
      const double P = (double)sel4(d, s.P[0], s.P[1], s.P[2], s.P[3]);
      double next;
      if (kExact) next = gather ? x * P : x / P;
      else next = gather ? x * P : divide_by_count(x, P, sel4(d, inverse[0], inverse[1], inverse[2], inverse[3]));
      x = j < place ? next : x;
    }
    if (gather) x = x * mine;
    const double t = x * coef;
    if (used && c < chunks) load = load + (twice ? t + t : t);
    if (c < chunks) emit(c, code);
  }
}

// The same where the NPU counts are powers of two (All-Reduces): the size before the
// lane's stage is an exponent less.  By four lanes that plan the same chunk each
// (plan_fast) it was 125 vector instructions a chunk, 20 to 27 % of a sweep on quads; 52 here
// (512-chunk sweep of 65,536 networks 27.9 -> 26.2 ms).
// emit(c, first, order): in every lane; first: the chunk starts on the lane's dimension.
template <typename Emit>
__device__ __forceinline__ void plan_quad_pow2(const Scenario& s, const FastScenario& fs, bool themis, bool rel,
                                               double thr, Emit emit) {
  const uint32_t k = threadIdx.x & 3u, D = (uint32_t)s.D;
  const bool used = k < D;
  const double coef = sel4((int)k, s.coef[0], s.coef[1], s.coef[2], s.coef[3]);
  const double fix = sel4((int)k, s.fix[0], s.fix[1], s.fix[2], s.fix[3]);
  const double below = rel ? thr * (fs.chunk * coef) : thr;   // the threshold where this dimension is the least loaded
  double load = used ? fix + fix : nan64();   // (no comparison with an unused dimension holds)
  // By the dimensions before this one (bit j + 2 of the place: k ^ j), 8 bits each: what this one
  // adds to the order's place (lexicographic: it counts the lower ones behind it, as many
  // times as the dimensions behind it have orders), and minus the sum of their log2 P.
  const bool lower1 = (k ^ 1u) < k, lower2 = (k ^ 2u) < k, lower3 = (k ^ 3u) < k;
  uint64_t weights = 0ull, less = 0ull;
  for (uint32_t m = 0; m < 8u; ++m) {
    uint32_t place = 0u, behind = 0u, sum = 0u;
#pragma unroll
    for (uint32_t j = 1; j < 4u; ++j) {
      const bool before = ((m >> (j - 1u)) & 1u) != 0u;
      place += before ? 1u : 0u;
      behind += (k ^ j) < k && !before ? 1u : 0u;
      sum += before ? (fs.epack >> (8u * (k ^ j))) & 0xffu : 0u;
    }
    const uint32_t left = place < D ? D - 1u - place : 0u;   // dimensions behind this one
    weights |= (uint64_t)(used ? behind * (left == 3u ? 6u : left) : 0u) << (8u * m);
    less |= (uint64_t)((0u - sum) & 0xffu) << (8u * m);
  }
  const uint32_t by_number = (lower1 ? 8u : 0u) | (lower2 ? 16u : 0u) | (lower3 ? 32u : 0u);
  for (uint32_t c = 0; c < s.C; ++c) {
    const double l1 = quad_other(load, 1u), l2 = quad_other(load, 2u), l3 = quad_other(load, 3u);
    // stable ascending order: an equal load goes first where its dimension is a lower one
    const bool lt1 = l1 < load, lt2 = l2 < load, lt3 = l3 < load;
    const bool eq1 = l1 == load, eq2 = l2 == load, eq3 = l3 == load;
    const uint32_t by_load = (lt1 || (lower1 && eq1) ? 8u : 0u) | (lt2 || (lower2 && eq2) ? 16u : 0u) |
                             (lt3 || (lower3 && eq3) ? 32u : 0u);
    const double lo = min_f64(min_f64(load, l1), min_f64(l2, l3)), hi = max_f64(max_f64(load, l1), max_f64(l2, l3));
    const bool within = hi - lo < below;   // (asked of the least loaded dimension)
    const bool sorts = used && by_load == 0u && !within;
    const uint32_t which = themis && quad_or(sorts ? 1u : 0u) != 0u ? by_load : by_number;
    const double t = ldexp(fs.chunk, (int)(int8_t)(less >> which)) * coef;
    load = __builtin_fma(2.0, t, load);   // (t + t is exact)
    emit(c, used && which == 0u, quad_sum((uint32_t)(weights >> which) & 0xffu));
  }
}

// One evaluation's queues on the lane's dimension, before the simulation: the
// chunks that start here, in the order of their ids.
template <typename L>
struct QuadQueue {
  uint8_t* block;
  uint32_t first = 0u, last = 0u;
  bool any = false;
  __device__ __forceinline__ explicit QuadQueue(void* lds) : block((uint8_t*)lds) {}
  __device__ __forceinline__ void add(uint32_t rec) {
    if (any) *L::link(block, last) = (uint16_t)rec;
    else first = rec;
    last = rec;
    any = true;
  }
};

struct QuadResult {
  double t_done;
  double busy;         // of the lane's dimension
  uint32_t started;    // operations of the lane's dimension
  bool ok;             // false: leave the evaluation to the follow-up passes
};

// The two event loops start 4 bytes behind a 32-byte line whatever comes before them: the
// place in the instruction stream is worth up to 4 % where a SIMD has few wavefronts, and
// moved with every change elsewhere (start modulo 32, us: 30,000 scenarios of 100 chunks
// 28 431, 8 413, 4 411; 20,001 of 250 chunks 20 1,021, 8 1,017, 4 1,005; sweep of 20,000
// with 200 chunks 16 3,315, 8 3,255, 4 3,206).
__device__ __forceinline__ void quad_loop_place() {
  asm volatile(".p2align 5\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0");
}

// What the lane's dimension has come to (see simulate_quad).
struct QuadRun {
  double f = nan64();      // finish time of the stage it serves, NaN when idle
  double busy = 0.0, now = 0.0;
  uint32_t sv = 0u;        // that stage, as the model passes it on
  uint32_t started = 0u;
  bool waits = false;      // chunks wait
};
// A pass up to the hand-over.  next: the earliest completion of the evaluation (NaN:
// nothing runs).  Returns the stage that is handed on; ending: the lanes whose stage ends now.
template <typename Model>
__device__ __forceinline__ uint32_t quad_hand_over(QuadRun& d, double next, uint64_t& ending) {
  // a8: the clock moves there
  d.now = max_f64(d.now, next);
  // of the stages that end now the one of the lowest chunk hands it on
  const bool ends = d.f == next;
  ending = __builtin_amdgcn_ballot_w64(ends);
  const uint32_t key = ends ? d.sv : Model::kNobody;
  const uint32_t given = quad_min_u32(key);
  if (ends && key == given) d.f = __hiloint2double(0x7ff80000, __double2loint(d.f));
  return given;
}
// Once all completions of the instant are delivered.  running: the lanes of the quads where
// something runs.
__device__ __forceinline__ bool quad_all_delivered(bool starts, uint64_t ending, uint64_t running) {
  if (__builtin_popcountll(ending) * 4 != __builtin_popcountll(running)) {   // more than one in some quad
    uint32_t mine = (uint32_t)(ending >> (threadIdx.x & 60u)) & 15u;
    asm volatile("" : "+v"(mine));   // (rare: a branch, not selects in every pass)
    starts = starts && (mine & (mine - 1u)) == 0u;
  }
  return starts;
}

// One class, first-in-first-out: a dimension's list is its first and its last record, in
// registers.  What a stage does depends on nothing that has to be read before, and the link
// behind its chunk is looked at a pass later, so a pass is one LDS trip and 45 vector
// instructions (the loop for any number of classes: two and 66).  65,536 3-D scenarios of
// 64 chunks, with the planner: 278 -> 234 us.
template <typename L, bool kPut, typename Model, typename Put>
__device__ __forceinline__ QuadRun quad_loop_fifo(const Model& model, const QuadQueue<L>& queue, Put put) {
  const uint32_t k = threadIdx.x & 3u;
  uint8_t* const block = queue.block;
  QuadRun d;
  uint32_t first = queue.first, last = queue.last;
  d.waits = queue.any;
  auto pass = [&](double next, uint64_t running) {
    uint64_t ending;
    const uint32_t given = quad_hand_over<Model>(d, next, ending);
    const bool append = model.goes_to(given, k);
    const uint32_t rec = Model::record(given);
    asm volatile("" : "+v"(first));   // (the wait for it: before the store, whose wait it would be as well)
    first = append && !d.waits ? rec : first;
    if (append && d.waits) *L::link(block, last) = (uint16_t)rec;
    last = append ? rec : last;
    d.waits = d.waits || append;
    if (quad_all_delivered(d.waits && !(d.f == d.f), ending, running)) {
      double time;
      bool turned;   // (never)
      const uint32_t link = *L::link(block, first);   // (only used where the list goes on)
      d.sv = model.template stage<true>(first, time, turned);
      d.f = d.now + time;
      d.busy = d.busy + time;
      if (kPut) put(d.started, (first & L::kIdMask) << 1 | ((first >> L::kPhaseBit) & 1u));
      ++d.started;
      d.waits = first != last;
      first = link;
    }
  };
  pass(nan64(), 0ull);
  quad_loop_place();
  // (every pass in which something runs completes a stage)
  for (uint32_t left = 2u * (uint32_t)kMaxDims * L::kCap + 16u; left != 0u; --left) {
    const double next = quad_min_f64(d.f);
    const uint64_t running = __builtin_amdgcn_ballot_w64(next == next);
    if (running == 0ull) break;
    pass(next, running);
  }
  return d;
}

// Any number of classes.
template <typename L, bool kPut, typename Model, typename Put>
__device__ __forceinline__ QuadRun quad_loop_classes(const Model& model, const QuadQueue<L>& queue, uint32_t cls0, Put put) {
  const uint32_t k = threadIdx.x & 3u;
  uint8_t* const block = queue.block;
  using Mask = typename std::conditional<(L::kPerDim > 32u), uint64_t, uint32_t>::type;
  // bit c: list of class c holds chunks; one bit behind the classes is always set, so that
  // there is a lowest one (the fourth: the place is in the banks of classes 3, 7, ..,
  // not in those of class 0, which is read the most)
  constexpr Mask kNone = (Mask)1 << (L::kPerDim + 3u);
  Mask lists = kNone;
  if (queue.any) {
    *L::ends(block, cls0) = queue.first | queue.last << 16;
    lists |= (Mask)1 << cls0;
  }
  QuadRun d;
  auto pass = [&](double next, uint64_t running) {
    uint64_t ending;
    const uint32_t given = quad_hand_over<Model>(d, next, ending);
    // (dimension 4, and that of kNobody where nothing ends: no lane's)
    const bool append = model.goes_to(given, k);
    const uint32_t to = Model::list(given);
    const Mask to_bit = (Mask)1 << to;
    const bool had = (lists & to_bit) != 0;
    if (append) lists |= to_bit;
    // an idle dimension with waiting chunks starts the first chunk of its lowest
    // class (smallest resident size), once all completions of the instant are delivered
    const bool starts = quad_all_delivered(!(d.f == d.f) && lists != kNone, ending, running);
    const uint32_t from = sizeof(Mask) == 8u ? (uint32_t)__builtin_ctzll(lists) : (uint32_t)__builtin_ctz((uint32_t)lists);
    typename L::Word* const from_at = L::ends(block, from);
    typename L::Word* const to_at = L::ends(block, to);
    uint32_t ends_from = *from_at, ends_to = *to_at;   // (either is used only where there is such a list)
    asm volatile("" : "+v"(ends_from), "+v"(ends_to));   // (read together, not each where it is needed)
    if (append) {
      const uint32_t rec = Model::record(given);
      if (had) *L::link(block, ends_to >> 16) = (uint16_t)rec;
      const uint32_t ends_now = __builtin_amdgcn_perm(rec, had ? ends_to : rec, 0x05040100u);
      *to_at = ends_now;
      if (to == from) ends_from = ends_now;
    }
    if (starts) {
      double time;
      bool turned;
      d.sv = model.template stage<false>(ends_from, time, turned);
      const uint32_t link = *L::link(block, ends_from);
      const bool last = ends_from == __builtin_amdgcn_alignbit(ends_from, ends_from, 16u);   // of its list
      lists &= last ? lists - 1u : ~(Mask)0;
      *(typename L::Half*)from_at = (uint16_t)link;   // (whatever it is where the list has ended)
      d.f = d.now + time;
      d.busy = d.busy + time;
      if (kPut) put(d.started, (ends_from & L::kIdMask) << 1 | ((ends_from >> L::kPhaseBit) & 1u));
      ++d.started;
      if (turned) {
        d.f = d.f + time;
        d.busy = d.busy + time;
        if (kPut) put(d.started, (ends_from & L::kIdMask) << 1 | 1u);
        ++d.started;
      }
    }
  };
  pass(nan64(), 0ull);
  quad_loop_place();
  for (uint32_t left = 2u * (uint32_t)kMaxDims * L::kCap + 16u; left != 0u; --left) {
    const double next = quad_min_f64(d.f);
    const uint64_t running = __builtin_amdgcn_ballot_w64(next == next);
    if (running == 0ull) break;
    pass(next, running);
  }
  d.waits = lists != kNone;
  return d;
}

// All four lanes of a quad call this with the same scenario and their own
// dimension's queue; cls0: the size class its chunks wait in.  Every lane of the
// wavefront has to be here (the quads exchange values with lane-crossing moves
// and leave the loop together), with `stages` = 0 where there is nothing to do.
// put(i, entry): the lane's dimension has started operation i (kPut).
template <typename L, bool kPut, typename Model, typename Put>
__device__ __forceinline__ QuadResult simulate_quad(const Model& model, QuadQueue<L>& queue, uint32_t cls0,
                                                    uint32_t stages, double t_min, Put put) {
  const QuadRun d = model.fifo ? quad_loop_fifo<L, kPut>(model, queue, put)
                               : quad_loop_classes<L, kPut>(model, queue, cls0, put);
  QuadResult res;
  res.t_done = d.now;
  res.busy = d.busy;
  res.started = d.started;
  // every stage ran and completed, and none was too short to move the clock, or for
  // the model
  const uint32_t settled = quad_min_u32(!(d.f == d.f) && !d.waits ? 1u : 0u);
  res.ok = quad_sum(d.started) == stages && settled != 0u && d.now < inf64() && d.now + 0.25 * t_min > d.now &&
           t_min >= Model::kShortest;
  return res;
}

}  // namespace themis
