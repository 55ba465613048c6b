// Queue simulation of traces with four lanes per trace: lane j of a quad owns
// dimension j (see themis_quad.hpp), sixteen traces to a wavefront; for large
// batches of traces released together on NPU counts that are powers of two.
//
// A batch that fills the GPU holds 64 traces per CU, 2.5 KiB of LDS each: the
// queues of one take 93 KB (200 collectives of 64 chunks on three dimensions), so
// they stay in memory, and what bounds an event is the chain of its instructions
// and waits.  With one lane per trace (themis_trace.hpp) a CU's 64 traces are one
// wavefront on one of its four SIMDs, whose event is 390 instructions and two
// dependent trips to memory; here they are four wavefronts, one per SIMD, an event
// is a third of the instructions, and no trip is waited for where it is made:
//   * a lane keeps the list of the lowest rank that holds chunks -- rank, first and
//     last record -- in registers, so a stage starts without reading memory, and
//     an append to that list is one store;
//   * the next record of that list, or the ends of the next list where it ran
//     empty, is asked for when a stage starts and looked at a pass later, as is
//     the size rank the chunk will have after the stage;
//   * an append behind another list's chunks waits a pass for that list's end.
// In LDS: per dimension which lists hold chunks (64 words of 64 bits at most, with a
// word in registers that says which are not zero), the collectives' chunk bytes,
// and the stage table.
//
// 16,384 traces of 200 collectives of 64 chunks on three dimensions: 139 -> 68 ms,
// some 2,050 clocks an event, half of them instructions and the rest the wait for
// what the last pass asked for (64 traces, whose queues are in the L2: 50 ms).
//
// Lists hold records, chunk << 6 | order + 32 * phase, and a link is the record of
// the next chunk.  The ends of a list whose records are in registers are stale in
// memory until a lower list takes its place.
#pragma once

#include "themis_quad.hpp"
#include "themis_trace.hpp"

namespace themis {

// LDS of a wavefront and a trace's region of the workspace, in bytes, for traces of
// up to D dimensions and Q collectives.
struct TraceQuadLayout {
  uint32_t lists;                      // per dimension
  uint32_t words, chunk, table, lds;   // (the bitmaps are at 0)
  uint32_t ends, ranks, region;        // (the links are at 0; the four dimensions' lists of a rank side by
                                       // side: they are in use at the same time, and share a line)
};
__host__ __device__ inline TraceQuadLayout trace_quad_layout(uint32_t slots, uint32_t D, uint32_t Q) {
  TraceQuadLayout l;
  l.lists = Q << D;
  l.words = (l.lists + 63u) / 64u;
  // (the collectives in the order of their chunks share the place of the bitmaps)
  l.chunk = 512u * l.words > 32u * Q ? 512u * l.words : 32u * Q;
  l.table = l.chunk + 128u * Q;
  l.lds = l.table + 1024u;
  l.ends = (4u * slots + 7u) & ~7u;
  l.ranks = l.ends + 32u * l.lists;
  l.region = l.ranks + 4u * l.lists;
  return l;
}

struct TraceQuadResult {
  double t_done, busy;
  uint32_t started;
  bool ok;
};

// All four lanes of a quad with the same trace; Q = 0 where there is none.  Every
// lane of the wavefront has to be here.  area: the regions of the wavefront's traces, stride apart.
// codes_at(q, c): the codes of chunks c .. c + 3 (a byte each), chunk_at(q); put(i, entry): the lane's dimension has
// started operation i.
template <bool kPut, typename CodesAt, typename ChunkAt, typename Put>
__device__ __forceinline__ TraceQuadResult simulate_trace_quad(const Scenario& s, const FastScenario& fs, uint32_t Q,
                                                               bool scf, double smallest, const TraceQuadLayout& l,
                                                               uint8_t* lds, uint8_t* area, uint32_t stride,
                                                               CodesAt codes_at, ChunkAt chunk_at, Put put) {
  const uint32_t k = threadIdx.x & 3u, quad = threadIdx.x >> 2, D = (uint32_t)s.D, C = s.C;
  const uint32_t masks = 1u << D;
  uint64_t* const bits = (uint64_t*)(lds + 8u * threadIdx.x);          // word w of the lane: bits[64 * w]
  uint16_t* const by_size = (uint16_t*)(lds + 2u * quad);              // position p: by_size[16 * p]
  double* const chunk = (double*)(lds + l.chunk + 8u * quad);          // collective q: chunk[16 * q]
  const uint8_t* const table = lds + l.table;
  // (byte offsets from the wavefront's area: an address in scalars and 32 bits per lane)
  const uint32_t links_at = quad * stride, ends_at = links_at + l.ends + 8u * k;
  const uint32_t ranks_at = links_at + l.ranks;
  typedef uint64_t __attribute__((aligned(4), may_alias)) Pair;
  typedef uint32_t __attribute__((may_alias)) Word;
  auto word = [&](uint32_t at) -> Word& { return *(Word*)(area + at); };
  auto pair = [&](uint32_t at) -> Pair& { return *(Pair*)(area + at); };
  auto link = [&](uint32_t rec) -> Word& { return word(links_at + ((rec >> 6) << 2)); };

#pragma unroll
  for (uint32_t j = 0; j < 4u; ++j)
    ((uint32_t*)(lds + l.table))[64u * j + threadIdx.x] = quad_stage_word(g_quad_stages, 64u * j + threadIdx.x);
  for (uint32_t q = k; q < Q; q += 4u) chunk[16u * q] = chunk_at(q);
  __syncthreads();

  // size ranks: the number of smaller sizes, counted by bisection in the
  // collectives' order for every mask (equal sizes share a rank)
  for (uint32_t q = k; q < Q; q += 4u) {
    const double v = chunk[16u * q];
    uint32_t at = 0u;
    for (uint32_t p = 0; p < Q; ++p) at += chunk[16u * p] < v || (chunk[16u * p] == v && p < q) ? 1u : 0u;
    by_size[16u * at] = (uint16_t)q;
  }
  __syncthreads();
  const uint32_t steps = 32u - (uint32_t)__clz((int)(Q | 1u));
  for (uint32_t at = k; at < Q * masks; at += 4u) {
    const uint32_t q = at / masks, m = at - q * masks;
    uint32_t smaller = 0u;
    if (scf) {
      const double v = chunk[16u * q];
      uint32_t lo[16], hi[16];
      double edge[16];
#pragma unroll
      for (uint32_t m2 = 0; m2 < 16u; ++m2) {
        lo[m2] = 0u;
        hi[m2] = m2 < masks ? Q : 0u;
        edge[m2] = ldexp(v, (int)esum(fs.epack, m2) - (int)esum(fs.epack, m));   // exact
      }
      // (eight searches side by side: their reads do not wait for each other)
#pragma unroll
      for (uint32_t half = 0; half < 16u; half += 8u) {
        if (half >= masks) break;
        for (uint32_t i = 0; i < steps; ++i) {
          uint32_t mid[8], who[8];
          double size[8];
#pragma unroll
          for (uint32_t j = 0; j < 8u; ++j) {
            mid[j] = (lo[half + j] + hi[half + j]) >> 1;
            who[j] = by_size[16u * min(mid[j], Q - 1u)];
          }
#pragma unroll
          for (uint32_t j = 0; j < 8u; ++j) size[j] = chunk[16u * who[j]];
#pragma unroll
          for (uint32_t j = 0; j < 8u; ++j) {
            const bool open = lo[half + j] < hi[half + j], below = size[j] < edge[half + j];
            lo[half + j] = open && below ? mid[j] + 1u : lo[half + j];
            hi[half + j] = open && !below ? mid[j] : hi[half + j];
          }
        }
      }
#pragma unroll
      for (uint32_t m2 = 0; m2 < 16u; ++m2) smaller += lo[m2];
    }
    word(ranks_at + 4u * at) = smaller;
  }
  __threadfence_block();
  __syncthreads();
  for (uint32_t w = 0; w < l.words; ++w) bits[64u * w] = 0ull;

  // a6: every chunk waits at the dimension of its first stage, collective by
  // collective; each lane takes the chunks that start on its own dimension
  uint64_t summary = 0ull;   // bit w: word w is not zero
  uint32_t bad = 0u;
  const uint32_t phase0 = fs.gather ? 32u : 0u;
  for (uint32_t q = 0; q < Q; ++q) {
    uint32_t first = 0u, last = 0u;
    bool any = false;
    for (uint32_t c4 = 0; c4 < C; c4 += 4u) {
      const uint32_t v = codes_at(q, c4);
      if (c4 + k < C && !order_code_ok((v >> (8u * k)) & 0xffu, s.D)) bad = 1u;
#pragma unroll
      for (uint32_t j = 0; j < 4u; ++j) {
        const uint32_t code = (v >> (8u * j)) & 0xffu;
        if (c4 + j < C && (code & 3u) == k) {
          const uint32_t order = (quad_row(D) + quad_order(stored_code(s, fs, code), D)) & 31u;
          const uint32_t rec = (q * C + c4 + j) << 6 | order | phase0;
          if (any) link(last) = rec;
          else first = rec;
          last = rec;
          any = true;
        }
      }
    }
    if (any && k < D) {
      const uint32_t r = word(ranks_at + 4u * (q * masks + (fs.state0 & 15u))), w = (r >> 6) & 63u;
      const uint64_t bit = 1ull << (r & 63u), had = bits[64u * w];
      if (had & bit) {
        const uint64_t e = pair(ends_at + 32u * r);
        link((uint32_t)(e >> 32)) = first;
        pair(ends_at + 32u * r) = (uint64_t)last << 32 | (uint32_t)e;
      } else {
        bits[64u * w] = had | bit;
        summary |= 1ull << w;
        pair(ends_at + 32u * r) = (uint64_t)last << 32 | first;
      }
    }
  }
  const bool malformed = quad_sum(bad) != 0u;
  if (malformed) summary = 0ull;

  double f = nan64(), busy = 0.0, now = 0.0;
  const double coef = sel4((int)k, s.coef[0], s.coef[1], s.coef[2], s.coef[3]);
  const double fix = sel4((int)k, s.fix[0], s.fix[1], s.fix[2], s.fix[3]);
  int less = 0;
#pragma unroll
  for (uint32_t d = 0; d < 4u; ++d) less |= (int)((0u - (fs.epack >> (8u * d) & 0xffu) & 0xffu) << (8u * d));
  // (a stand-alone All-Gather's sizes count from the full one)
  const int grown = fs.gather ? (int)fs.etot : 0;
  const uint32_t column = 4u * ((k + quad_column(D)) & 3u);
  const uint32_t wanted = fs.rs_only ? 7u | 32u << 3 : 7u;   // (see QuadPow2)
  uint32_t c_inv = (uint32_t)((0x80000000ull + C - 1u) / max(C, 1u));   // (an invalid trace may have none)
  asm volatile("" : "+v"(c_inv));   // (32 bits)
  constexpr uint32_t kNone = ~0u;
  const uint32_t last_word = l.words - 1u;
  uint32_t sv = 0u;                     // the running stage: record then << 3 | dimension it waits for (4: none)
  uint32_t rank_then = 0u;              // its size rank then
  uint32_t started = 0u;
  uint32_t low = kNone, head = 0u, tail = 0u;   // the lowest list (kNone: nothing waits)
  uint64_t asked = 0ull;                // what is on its way for it:
  uint32_t asked_for = 0u;              // 1: its first record, 2: both ends
  uint32_t behind = kNone, behind_rec = 0u, behind_tail = 0u;   // the append that waits for its list's end
  if (summary != 0ull) {
    const uint32_t w = (uint32_t)__builtin_ctzll(summary);
    low = w << 6 | (uint32_t)__builtin_ctzll(bits[64u * w]);
    asked = pair(ends_at + 32u * low);
    asked_for = 2u;
  }
  auto pass = [&](double next, uint64_t running) {
    now = max_f64(now, next);
    const bool stage_ends = f == next;
    const uint64_t ending = __builtin_amdgcn_ballot_w64(stage_ends);
    const uint32_t key = stage_ends ? sv : ~0u;
    const uint32_t given = quad_min_u32(key);
    const bool mine = stage_ends && key == given;
    if (mine) f = __hiloint2double(0x7ff80000, __double2loint(f));
    // what was asked for in the last pass
    const uint32_t r = quad_or(mine ? rank_then : 0u);
    if (asked_for != 0u) head = (uint32_t)asked;
    if (asked_for == 2u) tail = (uint32_t)(asked >> 32);
    asked_for = 0u;
    if (behind != kNone) {
      link(behind_tail) = behind_rec;
      if (behind == low) tail = behind_rec;
      else word(ends_at + 32u * behind + 4u) = behind_rec;
      behind = kNone;
    }
    // an idle dimension starts the first chunk of its lowest list, once all
    // completions of the instant are delivered
    bool can_start = !(f == f);
    if (__builtin_popcountll(ending) * 4 != __builtin_popcountll(running)) {
      uint32_t in_quad = (uint32_t)(ending >> (threadIdx.x & 60u)) & 15u;
      asm volatile("" : "+v"(in_quad));
      can_start = can_start && (in_quad & (in_quad - 1u)) == 0u;
    }
    // The chunk that is handed on joins the list of its rank, or is started at once
    // where that is below all others.  Everything that is read in LDS is read here,
    // together; a word that both the append and the start change is put right below.
    const bool append = (given & wanted) == k;
    const uint32_t rec = given >> 3;
    const bool lower = append && r < low;
    const bool starts = can_start && (lower || low != kNone), direct = starts && lower;
    const bool queued = append && !direct;
    const uint32_t begun = direct ? rec : head;
    const uint32_t q = __umulhi((begun >> 6) << 1, c_inv);
    // (some word where nothing waits)
    const uint32_t wr = (r >> 6) & 63u, wl = min(low >> 6, last_word);
    const uint64_t bit_r = 1ull << (r & 63u);
    const uint64_t all = queued ? summary | 1ull << wr : summary, others = all & ~(1ull << wl);
    const uint32_t w2 = min((uint32_t)__builtin_ctzll(others | 1ull << 63), last_word);
    uint32_t does = *(const uint32_t*)(table + ((begun & 63u) << 4 | column));
    double bytes = chunk[16u * q];
    uint64_t word_r = bits[64u * wr], word_l = bits[64u * wl], word_2 = bits[64u * w2];
    asm volatile("" : "+v"(does), "+v"(bytes), "+v"(word_r), "+v"(word_l), "+v"(word_2));
    summary = all;
    if (queued) {
      if (r == low) {
        link(tail) = rec;
        tail = rec;
      } else if ((word_r & bit_r) != 0ull) {   // its end is asked for
        behind = r;
        behind_rec = rec;
        behind_tail = word(ends_at + 32u * r + 4u);
      } else {
        bits[64u * wr] = word_r | bit_r;
        const uint32_t put_first = lower ? head : rec, put_last = lower ? tail : rec;
        if (low != kNone) pair(ends_at + 32u * max(r, low)) = (uint64_t)put_last << 32 | put_first;
        if (lower) {
          low = r;
          head = tail = rec;
        }
      }
    }
    if (starts) {
      rank_then = word(ranks_at + 4u * (q * masks + ((does >> 19) & 15u)));
      if (!direct) {
        // (one load for whichever it is, so that nothing waits for it here)
        uint32_t next_at = links_at + ((head >> 6) << 2);
        asked_for = 1u;
        if (head == tail) {
          const uint64_t in_word = (word_l & (word_l - 1ull)) | (queued && wr == wl ? bit_r : 0ull);
          const uint64_t in_next = word_2 | (queued && wr == w2 ? bit_r : 0ull);
          bits[64u * wl] = in_word;
          const uint64_t from = in_word != 0ull ? in_word : in_next;
          const uint32_t base = in_word != 0ull ? wl : w2;
          if (in_word == 0ull) summary = others;
          low = summary != 0ull ? base << 6 | (uint32_t)__builtin_ctzll(from) : kNone;
          next_at = low != kNone ? ends_at + 32u * low : next_at;
          asked_for = low != kNone ? 2u : 0u;   // (the head stays a record where nothing is left)
        }
        asked = pair(next_at);
      }
      double time = ldexp(bytes, __builtin_amdgcn_sdot4((int)(does & 0x01010101u), less, grown, false)) * coef;
      time = fix + time;
      sv = (begun >> 6) << 9 | ((does >> 9) & 63u) << 3 | ((does >> 1) & 7u);
      f = now + time;
      busy = busy + time;
      if (kPut) put(started, (begun >> 6) << 1 | ((begun >> 5) & 1u));
      ++started;
    }
  };
  pass(nan64(), 0ull);
  // (every pass in which something runs completes a stage)
  uint32_t most = (fs.rs_only || fs.gather ? D : 2u * D) * C * Q + 16u;
  for (int off = 32; off > 0; off >>= 1) most = max(most, (uint32_t)__shfl_xor((int)most, off));
  for (uint32_t left = (uint32_t)__builtin_amdgcn_readfirstlane((int)most); left != 0u; --left) {
    const double next = quad_min_f64(f);
    const uint64_t running = __builtin_amdgcn_ballot_w64(next == next);
    if (running == 0ull) break;
    pass(next, running);
  }
  TraceQuadResult res;
  res.t_done = now;
  res.busy = busy;
  res.started = started;
  // as in the other loops; the shortest stage there can be, at least
  double x = smallest;
  if (!fs.gather) x = ldexp(x, -(int)(fs.etot - (fs.epack >> (8u * k) & 0xffu)));
  const double shortest = quad_min_f64(k < D ? fix + x * coef : nan64());
  const uint32_t settled = quad_min_u32(!(f == f) && low == kNone ? 1u : 0u);
  const uint32_t stages = (fs.rs_only || fs.gather ? D : 2u * D) * C * Q;
  res.ok = !malformed && quad_sum(started) == stages && settled != 0u && now < inf64() &&
           now + 0.25 * shortest > now && shortest >= 2.2250738585072014e-308;
  return res;
}

}  // namespace themis
