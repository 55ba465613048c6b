// Queue simulation of a trace (several collectives of different sizes sharing
// the per-dimension queues) with a whole wavefront per trace, all of its state
// in registers and LDS: for batches of traces that do not fill the GPU with one
// lane each.
//
// What bounds a trace is the chain of its events, one after the other; with a
// lane per trace (themis_trace.hpp) an event of a lone wavefront is some 390
// instructions and two dependent trips to memory.  Here, as in
// themis_wave.hpp, everything an event decides is a scalar, so it executes only
// what it needs, and what it reads is in registers or one LDS trip away:
//   * the lists of a dimension -- one per resident size, up to 4,096 ranks --
//     that hold chunks are a bitmap in a register pair (lane = rank / 64, 64
//     bits each) with a 64-bit scalar that says which lanes have a bit set, so
//     the lowest rank is two searches for a first bit and two lane reads;
//   * first and last chunk per (dimension, rank), and per chunk its link (two
//     bytes) and state (one), are in LDS, as are the collectives' chunk sizes
//     and size ranks;
//   * what a stage does depends on the chunk's order and phase alone: tables
//     per dimension in registers, lane = rank of the order + 32 * phase.
// A chunk is named by twice its number, the byte offset of its link.
// An event is some 100 instructions and three LDS trips, 0.42 us on a lone
// wavefront (a lane per trace: 1.5 us, with release times 5); 2,001 traces of up
// to 50 collectives of 16 to 32 chunks with release times and queue orders: 36.9 ->
// 4.5 ms.  The other bound is the CU's LDS: 200 collectives of 64 chunks on three
// dimensions take 62 KiB (the links and states 38, the lists 19), two wavefronts.
//
// NPU counts that are not powers of two (kDivide): a stage's bytes are the
// chunk's, divided once per dimension reduced before, as divide_by_count() does.
#pragma once

#include "themis_generic.hpp"
#include "themis_trace.hpp"
#include "themis_wave.hpp"

namespace themis {

constexpr uint32_t kTraceWavePhase = 32u;          // lane = order rank + 32 * phase
// a running stage: chunk's name in bits 0-15, its state once the stage has
// ended in bits 16-21, the dimension it waits for then in bits 22-23, and
constexpr uint32_t kTraceWaveFinished = 1u << 24;  // whether it is finished
// (bits 0-11 of the table's entry: where its size rank is in the collective's row)

// Ranks of a collective's row: one per mask of reduced dimensions, or where
// divisions make the sizes, one per (dimension, phase, order).
__host__ __device__ inline uint32_t trace_wave_row(uint32_t D, bool by_order) {
  const uint32_t orders = D >= 4u ? 24u : D == 3u ? 6u : D;
  return by_order ? D * 2u * orders : 1u << D;
}
// Lists per dimension (ranks count sizes, so they stay below Q times the sizes
// of one collective; first-in-first-out has one list).
__host__ __device__ inline uint32_t trace_wave_lists(uint32_t D, uint32_t Q, bool scf, bool divide) {
  if (!scf) return 1u;
  return Q * (divide ? trace_wave_row(D, true) / D : 1u << D);
}
// LDS of one trace, in bytes.
struct TraceWaveLayout {
  uint32_t state, lists, records, release, order, bytes;   // offsets (the links are at 0)
  uint32_t record;   // bytes of a collective's record: its chunk's bytes (f64) and its size ranks (u16 each)
};
__host__ __device__ inline TraceWaveLayout trace_wave_layout(uint32_t slots, uint32_t D, uint32_t Q, bool scf,
                                                             bool divide) {
  TraceWaveLayout l;
  l.state = 2u * slots;
  l.lists = (l.state + slots + 7u) & ~7u;
  // (the sorted chunk sizes share the lists' place while the ranks are made)
  const uint32_t lists = 4u * D * trace_wave_lists(D, Q, scf, divide);
  l.records = l.lists + ((lists > 8u * Q ? lists : 8u * Q) + 7u) / 8u * 8u;
  l.record = (8u + 2u * trace_wave_row(D, scf && divide) + 7u) & ~7u;
  l.release = l.records + l.record * Q;
  l.order = l.release + 8u * Q;
  l.bytes = (l.order + 2u * Q + 15u) & ~15u;
  return l;
}

// One dimension of the event loop (values that are the same for all lanes: lane 0 of finish, busy and rank).
struct TraceWaveDim {
  double finish, busy;
  uint32_t running;            // the running stage, see above
  uint32_t started;            // operations so far
  uint64_t words;              // bit l: lane l of the bitmap is not zero
  uint32_t bits_lo, bits_hi;   // lists with chunks, lane = rank / 64
  uint32_t rank;               // size rank the running chunk has once its stage has ended
  uint32_t log;                // lane = operation number & 63: the last queue-order entries
};
struct TraceWaveTables {
  uint32_t bytes[kMaxDims];    // what turns the chunk's bytes into the stage's: a power of two, or
                               // the divisors (dimension + 1, three bits each)
  uint32_t next[kMaxDims];     // what the completion does
};

// The event loop, one assembly block for the reason given in themis_wave.hpp
// (whose wait states and shape it shares).  One lane is active; lane reads and
// writes do not look at that.
//
// K = dimension: fK finish, zK busy, rK running, cK started, wK words, eK / EK
// bitmap, kK rank, gK log, sK bytes, nK next, mK coefficient, aK delay, hK LDS
// address of the lists.
#define THEMIS_V_LOG_0(K)
#define THEMIS_V_LOG_1(K)                                                             \
  "s_bfe_u32 %[b], %[rc], 0x10015\n\t" "s_or_b32 %[b], %[b], %[id]\n\t"               \
  "s_mov_b32 m0, %[c" #K "]\n\t" "s_add_u32 %[c" #K "], %[c" #K "], 1\n\t"            \
  "v_writelane_b32 %[g" #K "], %[b], m0\n\t"                                          \
  "s_and_b32 %[b], %[c" #K "], 63\n\t"
#define THEMIS_V_FLUSH_0(K, E)
#define THEMIS_V_FLUSH_1(K, E) "s_cbranch_scc0 .Lvf" #E "_%=\n\t" ".Lvg" #E "_%=:\n\t"
#define THEMIS_V_START_AWAY_0(K, E)
// 64 entries to memory (rb: entries of a dimension's row, most: the bound that
// ends a loop whose records are broken)
#define THEMIS_V_START_AWAY_1(K, E)                                                   \
  ".Lvf" #E "_%=:\n\t" "s_cmp_gt_u32 %[c" #K "], %[rb]\n\t" "s_cbranch_scc1 .Lvend_%=\n\t" \
  "s_mul_i32 %[b], %[rb], " #K "\n\t" "s_add_u32 %[b], %[b], %[c" #K "]\n\t"          \
  "s_sub_u32 %[b], %[b], 64\n\t" "s_mov_b64 exec, -1\n\t"                             \
  "v_add_u32_e32 %[va], %[b], %[lane]\n\t"                                            \
  "s_cmp_eq_u32 %[wide], 0\n\t" "s_cbranch_scc1 .Lvy" #E "_%=\n\t"                    \
  "v_lshlrev_b32_e32 %[va], 1, %[va]\n\t"                                             \
  "global_store_short %[va], %[g" #K "], %[rows]\n\t" "s_mov_b64 exec, 1\n\t"         \
  "s_branch .Lvg" #E "_%=\n\t"                                                        \
  ".Lvy" #E "_%=:\n\t" "global_store_byte %[va], %[g" #K "], %[rows]\n\t" "s_mov_b64 exec, 1\n\t" \
  "s_branch .Lvg" #E "_%=\n\t"

// the bytes of the stage from the chunk's (vx), as bytes of the state (b) says
#define THEMIS_V_BYTES_0 "v_ldexp_f64 %[vx], %[vx], %[b]\n\t"
#define THEMIS_V_BYTES_1 "s_call_b64 vcc, .Lvdiv_%=\n\t"
#define THEMIS_V_DIVIDE_BY(K, L)                                                      \
  ".Lv" #L "_%=:\n\t" "s_cmp_lg_u32 %[gather], 0\n\t" "s_cbranch_scc1 .Lv" #L "g_%=\n\t" \
  "v_mul_f64 %[vt], %[vx], %[y" #K "]\n\t" "v_fma_f64 %[vx], -%[vt], %[P" #K "], %[vx]\n\t" \
  "v_fma_f64 %[vx], %[vx], %[y" #K "], %[vt]\n\t" "s_branch .Lvdiv_%=\n\t"            \
  ".Lv" #L "g_%=:\n\t" "v_mul_f64 %[vx], %[vx], %[P" #K "]\n\t" "s_branch .Lvdiv_%=\n\t"
#define THEMIS_V_DIVIDE_0
#define THEMIS_V_DIVIDE_1                                                             \
  ".Lvdiv_%=:\n\t" "s_and_b32 %[t], %[b], 7\n\t" "s_cbranch_scc0 .Lvdived_%=\n\t"     \
  "s_lshr_b32 %[b], %[b], 3\n\t"                                                      \
  "s_cmp_eq_u32 %[t], 2\n\t" "s_cbranch_scc1 .Lvd1_%=\n\t"                            \
  "s_cmp_eq_u32 %[t], 3\n\t" "s_cbranch_scc1 .Lvd2_%=\n\t"                            \
  "s_cmp_eq_u32 %[t], 4\n\t" "s_cbranch_scc1 .Lvd3_%=\n\t"                            \
  THEMIS_V_DIVIDE_BY(0, d0) THEMIS_V_DIVIDE_BY(1, d1) THEMIS_V_DIVIDE_BY(2, d2) THEMIS_V_DIVIDE_BY(3, d3) \
  ".Lvdived_%=:\n\t" "s_setpc_b64 vcc\n\t"

// chunk `id`: where the record of its collective is (q), and the read of its bytes
#define THEMIS_V_CHUNK                                                                \
  "s_mul_hi_u32 %[q], %[id], %[cinv]\n\t" "s_mul_i32 %[q], %[q], %[rsize]\n\t"        \
  "s_add_u32 %[q], %[q], %[rat]\n\t"                                                \
  "v_mov_b32_e32 %[va], %[q]\n\t" "ds_read_b64 %[vx], %[va]\n\t"
// its stage on K starts (the bytes are on their way), and the size rank it has
// afterwards is read
#define THEMIS_V_START(K, E, LOG, DIV)                                                \
  "s_lshr_b32 %[t], %[rc], 16\n\t"                                                  \
  "v_readlane_b32 %[b], %[s" #K "], %[t]\n\t" "v_readlane_b32 %[nx], %[n" #K "], %[t]\n\t" \
  "s_bitset0_b32 %[idle], " #K "\n\t" "s_waitcnt lgkmcnt(0)\n\t"                      \
  THEMIS_V_BYTES_##DIV                                                                \
  "s_and_b32 %[t], %[nx], 0xfff\n\t" "s_add_u32 %[t], %[t], %[q]\n\t"                 \
  "v_mul_f64 %[vx], %[vx], %[m" #K "]\n\t"                                            \
  "v_mov_b32_e32 %[va], %[t]\n\t" "ds_read_u16 %[k" #K "], %[va]\n\t"                 \
  "v_add_f64 %[vx], %[a" #K "], %[vx]\n\t"                                            \
  "s_and_b32 %[nx], %[nx], 0x1ff0000\n\t" "s_or_b32 %[r" #K "], %[id], %[nx]\n\t"     \
  THEMIS_V_LOG_##LOG(K)                                                               \
  "v_add_f64 %[f" #K "], %[now], %[vx]\n\t" "v_add_f64 %[z" #K "], %[z" #K "], %[vx]\n\t" \
  THEMIS_V_FLUSH_##LOG(K, E)

// the chunk of rc joins the list of rank vr of dimension N
#define THEMIS_V_PUSH(N, E)                                                           \
  "v_readfirstlane_b32 %[t], %[vr]\n\t" "s_and_b32 %[id], %[rc], 0xffff\n\t"          \
  "s_lshr_b32 %[c], %[t], 6\n\t" "s_and_b32 %[b], %[t], 63\n\t"                       \
  "v_readlane_b32 vcc_lo, %[e" #N "], %[c]\n\t" "v_readlane_b32 vcc_hi, %[E" #N "], %[c]\n\t" \
  "s_lshl2_add_u32 %[t], %[t], %[h" #N "]\n\t" "s_lshr_b32 %[nx], %[id], 1\n\t"       \
  "v_mov_b32_e32 %[va], %[t]\n\t" "s_add_u32 %[nx], %[nx], %[stat]\n\t"               \
  "s_lshr_b32 %[t], %[rc], 16\n\t" "v_mov_b32_e32 %[vb], %[nx]\n\t"                   \
  "v_mov_b32_e32 %[vd], %[t]\n\t" "v_mov_b32_e32 %[vr], %[id]\n\t"                    \
  "ds_write_b8 %[vb], %[vd]\n\t"                                                      \
  "s_bitcmp1_b64 vcc, %[b]\n\t" "s_cbranch_scc0 .Lve" #E "_%=\n\t"                    \
  "ds_read_u16 %[vd], %[va] offset:2\n\t" "ds_write_b16 %[va], %[vr] offset:2\n\t"    \
  "s_waitcnt lgkmcnt(1)\n\t" "ds_write_b16 %[vd], %[vr]\n\t" ".Lvp" #E "_%=:\n\t"
#define THEMIS_V_PUSH_AWAY(N, E)                                                      \
  ".Lve" #E "_%=:\n\t" "s_mov_b32 m0, %[c]\n\t" "s_pack_ll_b32_b16 %[t], %[id], %[id]\n\t" \
  "s_bitset1_b64 vcc, %[b]\n\t" "s_bitset1_b64 %[w" #N "], %[c]\n\t"                  \
  "v_writelane_b32 %[e" #N "], vcc_lo, m0\n\t" "v_writelane_b32 %[E" #N "], vcc_hi, m0\n\t" \
  "v_mov_b32_e32 %[vd], %[t]\n\t" "ds_write_b32 %[va], %[vd]\n\t" "s_branch .Lvp" #E "_%=\n\t"

// K takes the first chunk of its lowest list
#define THEMIS_V_PICK(K, E, DONE, LOG, DIV)                                           \
  "s_cmp_eq_u64 %[w" #K "], 0\n\t" "s_cbranch_scc1 " DONE "\n\t"                      \
  "s_ff1_i32_b64 %[c], %[w" #K "]\n\t" "s_mov_b32 m0, %[c]\n\t"                       \
  "v_readlane_b32 vcc_lo, %[e" #K "], %[c]\n\t" "v_readlane_b32 vcc_hi, %[E" #K "], %[c]\n\t" \
  "s_lshl_b32 %[t], %[c], 8\n\t" "s_add_u32 %[t], %[t], %[h" #K "]\n\t"               \
  "s_ff1_i32_b64 %[b], vcc\n\t" "s_lshl2_add_u32 %[t], %[b], %[t]\n\t"                \
  "v_mov_b32_e32 %[vr], %[t]\n\t" "ds_read_b32 %[vd], %[vr]\n\t"                      \
  "s_waitcnt lgkmcnt(0)\n\t" "v_readfirstlane_b32 %[nx], %[vd]\n\t"                   \
  "s_and_b32 %[id], %[nx], 0xffff\n\t" "s_lshr_b32 %[t], %[id], 1\n\t"                \
  "s_add_u32 %[t], %[t], %[stat]\n\t" "v_mov_b32_e32 %[vb], %[id]\n\t"                \
  "v_mov_b32_e32 %[va], %[t]\n\t" "ds_read_u8 %[va], %[va]\n\t" "ds_read_u16 %[vb], %[vb]\n\t" \
  "s_lshr_b32 %[nx], %[nx], 16\n\t" "s_cmp_eq_u32 %[nx], %[id]\n\t"                   \
  "s_cbranch_scc1 .Lvl" #E "_%=\n\t"                                                  \
  "s_waitcnt lgkmcnt(0)\n\t" "ds_write_b16 %[vr], %[vb]\n\t" ".Lvs" #E "_%=:\n\t"     \
  "v_readfirstlane_b32 %[rc], %[va]\n\t" THEMIS_V_CHUNK                               \
  "s_lshl_b32 %[rc], %[rc], 16\n\t" THEMIS_V_START(K, E, LOG, DIV)
// (out of line: it was the list's last chunk)
#define THEMIS_V_PICK_AWAY(K, E, LOG)                                                 \
  ".Lvl" #E "_%=:\n\t" "s_bitset0_b64 vcc, %[b]\n\t" "s_cmp_eq_u64 vcc, 0\n\t"        \
  "s_cselect_b32 %[nx], 1, 0\n\t"                                                     \
  "v_writelane_b32 %[e" #K "], vcc_lo, m0\n\t" "v_writelane_b32 %[E" #K "], vcc_hi, m0\n\t" \
  "s_bfm_b64 vcc, %[nx], %[c]\n\t" "s_andn2_b64 %[w" #K "], %[w" #K "], vcc\n\t"      \
  "s_waitcnt lgkmcnt(0)\n\t" "s_branch .Lvs" #E "_%=\n\t" THEMIS_V_START_AWAY_##LOG(K, E)

// the stage on K has ended alone at this instant, its chunk goes to N: at once
// where N is idle
#define THEMIS_V_HAND_ON(K, N)                                                        \
  ".Lvt" #K #N "_%=:\n\t" "s_bitset1_b32 %[idle], " #K "\n\t"                         \
  "s_bitcmp1_b32 %[idle], " #N "\n\t" "s_cbranch_scc1 .Lvh" #K #N "_%=\n\t"           \
  THEMIS_V_PUSH(N, K##N) "s_branch .Lvk" #K "_%=\n\t"
#define THEMIS_V_HAND_ON_AWAY(K, N, LOG, DIV)                                         \
  THEMIS_V_PUSH_AWAY(N, K##N)                                                         \
  ".Lvh" #K #N "_%=:\n\t" "s_and_b32 %[id], %[rc], 0xffff\n\t" THEMIS_V_CHUNK         \
  THEMIS_V_START(N, d##K##N, LOG, DIV) "s_branch .Lvk" #K "_%=\n\t"                   \
  THEMIS_V_START_AWAY_##LOG(N, d##K##N)
#define THEMIS_V_ENDED(K, A, B, C, LOG, DIV)                                          \
  ".Lvc" #K "_%=:\n\t"                                                                \
  "s_and_b32 %[rc], %[r" #K "], 0x3fffff\n\t" "v_mov_b64_e32 %[f" #K "], %[nan]\n\t"  \
  "s_bitcmp1_b32 %[r" #K "], 24\n\t" "s_cbranch_scc1 .Lvi" #K "_%=\n\t"               \
  "s_lshr_b32 %[t], %[r" #K "], 22\n\t" "s_waitcnt lgkmcnt(0)\n\t" "v_mov_b32_e32 %[vr], %[k" #K "]\n\t" \
  "s_cmp_eq_u32 %[t], " #A "\n\t" "s_cbranch_scc1 .Lvt" #K #A "_%=\n\t"               \
  "s_cmp_eq_u32 %[t], " #B "\n\t" "s_cbranch_scc1 .Lvt" #K #B "_%=\n\t"               \
  "s_cmp_eq_u32 %[t], " #C "\n\t" "s_cbranch_scc1 .Lvt" #K #C "_%=\n\t"               \
  THEMIS_V_PUSH(K, K##K)                                                              \
  ".Lvi" #K "_%=:\n\t" "s_bitset1_b32 %[idle], " #K "\n\t"                            \
  ".Lvk" #K "_%=:\n\t" THEMIS_V_PICK(K, K, ".Lvnext_%=", LOG, DIV) "s_branch .Lvnext_%=\n\t" \
  THEMIS_V_HAND_ON(K, A) THEMIS_V_HAND_ON(K, B) THEMIS_V_HAND_ON(K, C)                \
  THEMIS_V_PUSH_AWAY(K, K##K) THEMIS_V_PICK_AWAY(K, K, LOG)                           \
  THEMIS_V_HAND_ON_AWAY(K, A, LOG, DIV) THEMIS_V_HAND_ON_AWAY(K, B, LOG, DIV)         \
  THEMIS_V_HAND_ON_AWAY(K, C, LOG, DIV)

// several at one instant: lowest chunk first, then every idle dimension takes its next
#define THEMIS_V_LOWEST(K)                                                            \
  "s_and_b32 %[t], %[r" #K "], 0xffff\n\t" "s_bitcmp1_b32 %[ends], " #K "\n\t"        \
  "s_cselect_b32 %[t], %[t], -1\n\t" "s_min_u32 %[nx], %[nx], %[t]\n\t"
#define THEMIS_V_IS_LOWEST(K)                                                         \
  "s_bitcmp1_b32 %[ends], " #K "\n\t" "s_cbranch_scc0 .Lvn" #K "_%=\n\t"              \
  "s_and_b32 %[t], %[r" #K "], 0xffff\n\t" "s_cmp_eq_u32 %[t], %[nx]\n\t"             \
  "s_cbranch_scc0 .Lvn" #K "_%=\n\t"                                                  \
  "s_mov_b32 %[rc], %[r" #K "]\n\t" "v_mov_b64_e32 %[f" #K "], %[nan]\n\t"            \
  "v_mov_b32_e32 %[vr], %[k" #K "]\n\t"                                               \
  "s_bitset0_b32 %[ends], " #K "\n\t" "s_bitset1_b32 %[idle], " #K "\n\t"             \
  "s_branch .Lvmd_%=\n\t" ".Lvn" #K "_%=:\n\t"
#define THEMIS_V_TAKE_TURN(K, LOG, DIV)                                               \
  "s_bitcmp1_b32 %[idle], " #K "\n\t" "s_cbranch_scc0 .Lva" #K "_%=\n\t"              \
  THEMIS_V_PICK(K, a##K, ".Lva" #K "_%=", LOG, DIV) ".Lva" #K "_%=:\n\t"
#define THEMIS_V_SEVERAL(LOG, DIV)                                                    \
  ".Lvm_%=:\n\t" "s_waitcnt lgkmcnt(0)\n\t" "s_mov_b32 %[nx], -1\n\t"                 \
  THEMIS_V_LOWEST(0) THEMIS_V_LOWEST(1) THEMIS_V_LOWEST(2) THEMIS_V_LOWEST(3)         \
  THEMIS_V_IS_LOWEST(0) THEMIS_V_IS_LOWEST(1) THEMIS_V_IS_LOWEST(2) THEMIS_V_IS_LOWEST(3) \
  "s_branch .Lvend_%=\n\t"                                                            \
  ".Lvmd_%=:\n\t" "s_bitcmp1_b32 %[rc], 24\n\t" "s_cbranch_scc1 .Lvmn_%=\n\t"         \
  "s_lshr_b32 %[t], %[rc], 22\n\t" "s_and_b32 %[rc], %[rc], 0x3fffff\n\t"             \
  "s_cmp_eq_u32 %[t], 0\n\t" "s_cbranch_scc1 .Lvm0_%=\n\t"                            \
  "s_cmp_eq_u32 %[t], 1\n\t" "s_cbranch_scc1 .Lvm1_%=\n\t"                            \
  "s_cmp_eq_u32 %[t], 2\n\t" "s_cbranch_scc1 .Lvm2_%=\n\t"                            \
  THEMIS_V_PUSH(3, m3) "s_branch .Lvmn_%=\n\t"                                        \
  ".Lvm0_%=:\n\t" THEMIS_V_PUSH(0, m0) "s_branch .Lvmn_%=\n\t"                        \
  ".Lvm1_%=:\n\t" THEMIS_V_PUSH(1, m1) "s_branch .Lvmn_%=\n\t"                        \
  ".Lvm2_%=:\n\t" THEMIS_V_PUSH(2, m2)                                                \
  ".Lvmn_%=:\n\t" "s_cmp_lg_u32 %[ends], 0\n\t" "s_cbranch_scc1 .Lvm_%=\n\t"          \
  ".Lvall_%=:\n\t" THEMIS_V_TAKE_TURN(0, LOG, DIV) THEMIS_V_TAKE_TURN(1, LOG, DIV)    \
  THEMIS_V_TAKE_TURN(2, LOG, DIV) THEMIS_V_TAKE_TURN(3, LOG, DIV) "s_branch .Lvnext_%=\n\t" \
  THEMIS_V_PUSH_AWAY(0, m0) THEMIS_V_PUSH_AWAY(1, m1) THEMIS_V_PUSH_AWAY(2, m2) THEMIS_V_PUSH_AWAY(3, m3) \
  THEMIS_V_PICK_AWAY(0, a0, LOG) THEMIS_V_PICK_AWAY(1, a1, LOG)                       \
  THEMIS_V_PICK_AWAY(2, a2, LOG) THEMIS_V_PICK_AWAY(3, a3, LOG)

// until the earliest completion does not come before the next release (rel;
// infinite, or nothing runs: the end)
#define THEMIS_V_LOOP(LOG, DIV)                                                       \
  "s_nop 4\n\t" "s_mov_b64 exec, 1\n\t" "s_nop 4\n\t" "s_branch .Lvall_%=\n\t"        \
  ".Lvnext_%=:\n\t"                                                                   \
  "v_min_f64 %[vt], %[f0], %[f1]\n\t" "v_min_f64 %[vx], %[f2], %[f3]\n\t"             \
  "v_min_f64 %[vt], %[vt], %[vx]\n\t"                                                 \
  "v_cmp_lt_f64_e64 vcc, %[vt], %[rel]\n\t" "v_cmp_eq_f64_e64 %[e0_], %[f0], %[vt]\n\t" \
  "v_cmp_eq_f64_e64 %[e1_], %[f1], %[vt]\n\t" "v_cmp_eq_f64_e64 %[e2_], %[f2], %[vt]\n\t" \
  "v_cmp_eq_f64_e64 %[e3_], %[f3], %[vt]\n\t"                                         \
  "s_and_b64 vcc, vcc, 1\n\t" "s_cbranch_scc0 .Lvend_%=\n\t"                          \
  "s_lshl_b64 %[e1_], %[e1_], 1\n\t" "s_lshl_b64 %[e2_], %[e2_], 2\n\t"               \
  "s_or_b64 %[e0_], %[e0_], %[e1_]\n\t" "s_lshl_b64 %[e3_], %[e3_], 3\n\t"            \
  "s_or_b64 %[e2_], %[e2_], %[e3_]\n\t" "s_or_b64 vcc, %[e0_], %[e2_]\n\t"            \
  "v_mov_b64_e32 %[now], %[vt]\n\t"                                                   \
  "s_sub_u32 %[passes], %[passes], 1\n\t" "s_cbranch_scc1 .Lvend_%=\n\t"              \
  "s_and_b32 %[ends], vcc_lo, 15\n\t" "s_add_u32 %[t], %[ends], -1\n\t"               \
  "s_and_b32 %[t], %[t], %[ends]\n\t" "s_cbranch_scc1 .Lvm_%=\n\t"                    \
  "s_cmp_gt_u32 %[ends], 2\n\t" "s_cbranch_scc1 .Lv23_%=\n\t"                         \
  "s_bitcmp1_b32 %[ends], 1\n\t" "s_cbranch_scc1 .Lvc1_%=\n\t"                        \
  THEMIS_V_ENDED(0, 1, 2, 3, LOG, DIV) THEMIS_V_ENDED(1, 0, 2, 3, LOG, DIV)           \
  ".Lv23_%=:\n\t" "s_bitcmp1_b32 %[ends], 3\n\t" "s_cbranch_scc1 .Lvc3_%=\n\t"        \
  THEMIS_V_ENDED(2, 0, 1, 3, LOG, DIV) THEMIS_V_ENDED(3, 0, 1, 2, LOG, DIV)           \
  THEMIS_V_SEVERAL(LOG, DIV) THEMIS_V_DIVIDE_##DIV                                    \
  ".Lvend_%=:\n\t" "s_mov_b64 exec, -1\n\t" "s_waitcnt lgkmcnt(0)\n\t" "s_nop 4\n\t"

#define THEMIS_V_DIM(K)                                                               \
  [f##K] "+&v"(d[K].finish), [z##K] "+&v"(d[K].busy), [e##K] "+&v"(d[K].bits_lo), [E##K] "+&v"(d[K].bits_hi), \
  [k##K] "+&v"(d[K].rank), [g##K] "+&v"(d[K].log), [r##K] "+&s"(d[K].running), [w##K] "+&s"(d[K].words), \
  [c##K] "+&s"(d[K].started)
#define THEMIS_V_TABLE(K)                                                             \
  [s##K] "v"(t.bytes[K]), [n##K] "v"(t.next[K]), [m##K] "v"(s.coef[K]), [a##K] "v"(s.fix[K]), [h##K] "s"(list_at[K])
#define THEMIS_V_DIVISOR(K) [P##K] "v"(divisor[K]), [y##K] "v"(inverse[K])

// What the loop keeps between two calls (a release lies between them).
struct TraceWaveRun {
  double now;
  uint32_t idle, passes;   // (passes: every one completes a stage; the bound ends the loop)
};

// rows: queue orders of the trace (kLog), `row_len` entries per dimension.
// Returns the earliest completion that is still to come (NaN: nothing runs).
template <bool kLog, bool kDivide>
__device__ __forceinline__ double trace_wave_events(const Scenario& s, const TraceWaveTables& t,
                                                    TraceWaveDim (&d)[kMaxDims], TraceWaveRun& run, double rel,
                                                    uint32_t c_inv, uint32_t record_at, uint32_t record_bytes,
                                                    uint32_t state_at,
                                                    const uint32_t (&list_at)[kMaxDims], uint32_t gather,
                                                    const double (&divisor)[kMaxDims],
                                                    const double (&inverse)[kMaxDims], void* rows,
                                                    uint32_t row_len, uint32_t wide) {
  double vt, vx;
  uint32_t rc, nx, tmp, cls, bit, id, q, ends, va, vb, vd, vr;
  uint64_t e0, e1, e2, e3;
  const uint32_t lane = lane_id();
#define THEMIS_V_RUN(LOG, DIV, ...)                                                   \
  asm volatile(THEMIS_V_LOOP(LOG, DIV)                                                \
      : THEMIS_V_DIM(0), THEMIS_V_DIM(1), THEMIS_V_DIM(2), THEMIS_V_DIM(3),           \
        [now] "+&v"(run.now), [vt] "=&v"(vt), [vx] "=&v"(vx), [va] "=&v"(va), [vb] "=&v"(vb), [vd] "=&v"(vd), \
        [vr] "=&v"(vr), [idle] "+&s"(run.idle), [passes] "+&s"(run.passes), [rc] "=&s"(rc), [nx] "=&s"(nx), \
        [t] "=&s"(tmp), [c] "=&s"(cls), [b] "=&s"(bit), [id] "=&s"(id), [q] "=&s"(q), [ends] "=&s"(ends), \
        [e0_] "=&s"(e0), [e1_] "=&s"(e1), [e2_] "=&s"(e2), [e3_] "=&s"(e3)            \
      : THEMIS_V_TABLE(0), THEMIS_V_TABLE(1), THEMIS_V_TABLE(2), THEMIS_V_TABLE(3),   \
        [nan] "v"(nan64()), [rel] "v"(rel), [cinv] "s"(c_inv), [rsize] "s"(record_bytes), [rat] "s"(record_at), \
        [stat] "s"(state_at) __VA_ARGS__                                              \
      : "vcc", "scc", "memory")
#define THEMIS_V_ROWS , [rows] "s"(rows), [rb] "s"(row_len), [wide] "s"(wide), [lane] "v"(lane)
#define THEMIS_V_DIVISORS \
  , [gather] "s"(gather), THEMIS_V_DIVISOR(0), THEMIS_V_DIVISOR(1), THEMIS_V_DIVISOR(2), THEMIS_V_DIVISOR(3)
  if constexpr (kLog && kDivide) THEMIS_V_RUN(1, 1, THEMIS_V_ROWS THEMIS_V_DIVISORS);
  else if constexpr (kLog) THEMIS_V_RUN(1, 0, THEMIS_V_ROWS);
  else if constexpr (kDivide) THEMIS_V_RUN(0, 1, THEMIS_V_DIVISORS);
  else THEMIS_V_RUN(0, 0);
#undef THEMIS_V_RUN
#undef THEMIS_V_ROWS
#undef THEMIS_V_DIVISORS
  return lane_get(vt, 0u);
}

__device__ __forceinline__ uint64_t first_lane(uint64_t v) {
  return (uint64_t)first_lane((uint32_t)(v >> 32)) << 32 | first_lane((uint32_t)v);
}

// Where the size rank of a chunk is in its collective's record (bytes): it waits
// for dimension k in phase `phase`, `mask` its reduced dimensions, r the rank of its order.
__device__ __forceinline__ uint32_t trace_wave_rank_at(bool by_order, uint32_t D, uint32_t mask, uint32_t k,
                                                       uint32_t phase, uint32_t r) {
  // the order's place among those of D dimensions (ring_order_rank is of four)
  const uint32_t orders = factorial_u32(D);
  const uint32_t at = D >= 4u ? r : D == 3u ? r / 6u * 2u + r % 6u / 2u : r / 6u;
  return 8u + 2u * (by_order ? (k * 2u + phase) * orders + at : mask);
}

// One trace, all 64 lanes with the same arguments (Q collectives of s.C chunks;
// kDivide: halvings are not exact, but no size leaves the normal range).  LDS
// from offset 0 on, as the layout says.  code_at(q, c): order code; chunk_at(q):
// bytes of a chunk; smallest: the least of those.
template <bool kLog, bool kDivide, typename CodeAt, typename ChunkAt, typename ReleaseAt>
__device__ __forceinline__ WaveOutcome trace_wave_simulate(const Scenario& s, uint32_t Q, bool scf,
                                                           bool has_release, double smallest,
                                                           const TraceWaveLayout& l, uint8_t* lds,
                                                           CodeAt code_at, ChunkAt chunk_at,
                                                           ReleaseAt release_at, void* rows, uint32_t row_len,
                                                           uint32_t wide, WaveResult& r) {
  const uint32_t lane = lane_id(), D = (uint32_t)s.D, C = s.C, G = Q * C;
  const bool gather = s.ctype == THEMIS_COLL_ALL_GATHER, rs_only = s.ctype == THEMIS_COLL_REDUCE_SCATTER;
  const uint32_t full = (1u << D) - 1u;
  const bool by_order = kDivide && scf;
  uint16_t* const link = (uint16_t*)lds;
  uint8_t* const state = lds + l.state;
  uint32_t* const lists = (uint32_t*)(lds + l.lists);
  double* const sorted = (double*)(lds + l.lists);
  double* const release = (double*)(lds + l.release);
  uint16_t* const order = (uint16_t*)(lds + l.order);
  auto chunk_of = [&](uint32_t q) -> double& { return *(double*)(lds + l.records + q * l.record); };
  auto rank_of = [&](uint32_t q, uint32_t at) -> uint16_t& {
    return *(uint16_t*)(lds + l.records + q * l.record + at);
  };

  bool bad = false;
  for (uint32_t g = lane; g < G; g += 64u) {
    const uint32_t q = g / C, code = code_at(q, g - q * C);
    bad = bad || !order_code_ok(code, s.D);
    state[g] = (uint8_t)(ring_order_rank(gather ? reverse_code(code, s.D) : code, D) % kWaveOrders +
                         (gather ? kTraceWavePhase : 0u));
  }
  if (uniform(bad)) return WaveOutcome::kMalformed;
  for (uint32_t q = lane; q < Q; q += 64u) {
    chunk_of(q) = chunk_at(q);
    if (has_release) release[q] = release_at(q);
    for (uint32_t m = 0; m < (l.record - 8u) / 2u; ++m) rank_of(q, 8u + 2u * m) = 0u;
  }
  __syncthreads();

  // collectives in the order of their releases (ties: by number)
  for (uint32_t q = lane; q < Q; q += 64u) {
    uint32_t at = q;
    if (has_release) {
      const double v = release[q];
      at = 0u;
      for (uint32_t p = 0; p < Q; ++p) at += release[p] < v || (release[p] == v && p < q) ? 1u : 0u;
      sorted[at] = v;
    }
    order[at] = (uint16_t)q;
  }
  __syncthreads();
  if (has_release)
    for (uint32_t q = lane; q < Q; q += 64u) release[q] = sorted[q];
  __syncthreads();

  // Size ranks: the number of smaller sizes among those that can wait (equal
  // sizes share a rank).  The collectives' sizes under one mask (division mode:
  // in one phase of one order) are in the order of their chunks, so the smaller
  // ones are counted by bisection.
  if (scf) {
    for (uint32_t q = lane; q < Q; q += 64u) {
      const double v = chunk_of(q);
      uint32_t at = 0u;
      for (uint32_t p = 0; p < Q; ++p) at += chunk_of(p) < v || (chunk_of(p) == v && p < q) ? 1u : 0u;
      sorted[at] = v;
    }
    __syncthreads();
    if constexpr (!kDivide) {
      uint32_t e[kMaxDims];
      for (int k = 0; k < kMaxDims; ++k) e[k] = k < s.D ? 31u - (uint32_t)__clz((int)s.P[k]) : 0u;
      auto esum_of = [&](uint32_t m) {
        return (int)((m & 1u ? e[0] : 0u) + (m & 2u ? e[1] : 0u) + (m & 4u ? e[2] : 0u) + (m & 8u ? e[3] : 0u));
      };
      const uint32_t steps = 32u - (uint32_t)__clz((int)Q);   // of a bisection of Q places
      for (uint32_t at = lane; at < Q << D; at += 64u) {
        const uint32_t q = at >> D, m = at & full;
        const double v = chunk_of(q);
        uint32_t smaller = 0u;
        for (uint32_t m2 = 0; m2 <= full; ++m2) {
          const double edge = ldexp(v, esum_of(m2) - esum_of(m));   // exact
          uint32_t lo = 0u, hi = Q;
          for (uint32_t i = 0; i < steps; ++i) {
            const uint32_t mid = (lo + hi) >> 1;
            const bool below = lo < hi && sorted[min(mid, Q - 1u)] < edge;
            if (below) lo = mid + 1u;
            else if (lo < hi) hi = mid;
          }
          smaller += lo;
        }
        rank_of(q, 8u + 2u * m) = (uint16_t)smaller;
      }
    } else {
      const uint32_t F = factorial_u32(D);
      auto place_of = [&](uint32_t code, uint32_t k) {
        uint32_t place = 0u;
        for (uint32_t j = 0; j < D; ++j) place = ((code >> (2u * j)) & 3u) == k ? j : place;
        return place;
      };
      for (uint32_t at = lane; at < Q * D * 2u * F; at += 64u) {
        const uint32_t q = at / (D * 2u * F), in = at - q * (D * 2u * F);
        const uint32_t k = in / (2u * F), phase = in / F & 1u;
        if (phase ? rs_only : gather) continue;
        const uint32_t code = nth_permutation_code(D, in % F);
        const double v = trace_resident_bytes(s, chunk_of(q), code, place_of(code, k), phase, gather);
        uint32_t smaller = 0u;
        for (uint32_t ph = gather ? 1u : 0u; ph < (rs_only ? 1u : 2u); ++ph)
          for (uint32_t f = 0; f < F; ++f) {
            const uint32_t c2 = nth_permutation_code(D, f), p2 = place_of(c2, k);
            uint32_t lo = 0u, hi = Q;
            while (lo < hi) {
              const uint32_t mid = (lo + hi) >> 1;
              if (trace_resident_bytes(s, sorted[mid], c2, p2, ph, gather) < v) lo = mid + 1u;
              else hi = mid;
            }
            smaller += lo;
          }
        rank_of(q, 8u + 2u * in) = (uint16_t)smaller;
      }
    }
    __syncthreads();
  }

  // tables, lane = order rank + 32 * phase
  TraceWaveTables t;
  const uint32_t phase = lane / kTraceWavePhase;
  const uint32_t rank = min(lane % kTraceWavePhase, kWaveOrders - 1u);
  const uint32_t code = ring_order_of_rank(rank);
  for (int k = 0; k < kMaxDims; ++k) t.bytes[k] = t.next[k] = 0u;
  {
    uint32_t mask = 0u, seq = 0u;
    int before = 0;
    for (uint32_t j = 0; j < D; ++j) {
      const uint32_t place = gather ? D - 1u - j : j;   // a stand-alone All-Gather grows from the last field on
      const uint32_t kj = (code >> (2u * place)) & 3u;
      const int ej = 31 - __clz(sel4((int)kj, (int)s.P[0], (int)s.P[1], (int)s.P[2], (int)s.P[3]));
      if (gather) {
        before += ej;
        seq |= (kj + 1u) << (3u * j);
      }
#pragma unroll
      for (uint32_t k = 0; k < (uint32_t)kMaxDims; ++k)
        if (k == kj) t.bytes[k] = kDivide ? seq : (uint32_t)before;
      if (!gather) {
        before -= ej;
        seq |= (kj + 1u) << (3u * j);
      }
    }
    for (uint32_t j = 0; j < D; ++j) {
      const uint32_t kj = (code >> (2u * j)) & 3u;
      const uint32_t upto = mask;   // the dimensions before kj
      mask |= 1u << kj;
      uint32_t to = kj, ph = phase, m = mask;
      bool fin = false;
      if (phase == 0u) {
        if (j + 1u == D) { fin = rs_only; ph = 1u; }
        else to = (code >> (2u * (j + 1u))) & 3u;
      } else {
        m = upto;
        if (j == 0u) fin = true;
        else to = (code >> (2u * (j - 1u))) & 3u;
      }
      const uint32_t next = trace_wave_rank_at(by_order, D, fin ? 0u : m, to, fin && !gather ? 0u : ph, rank) |
                            (rank + kTraceWavePhase * ph) << 16 | to << 22 | (fin ? kTraceWaveFinished : 0u);
#pragma unroll
      for (uint32_t k = 0; k < (uint32_t)kMaxDims; ++k)
        if (k == kj) t.next[k] = next;
    }
  }
  // where a chunk waits first, and its size rank there
  const uint32_t first_dim = (code >> (gather ? 2u * (D - 1u) : 0u)) & 3u;
  const uint32_t first_at = trace_wave_rank_at(by_order, D, gather ? full : 0u, first_dim, gather ? 1u : 0u, rank);

  TraceWaveDim d[kMaxDims];
  uint32_t list_at[kMaxDims];
  const uint32_t per_dim = trace_wave_lists(D, Q, scf, kDivide);
#pragma unroll
  for (uint32_t k = 0; k < (uint32_t)kMaxDims; ++k) {
    d[k].finish = nan64();
    d[k].busy = 0.0;
    d[k].running = d[k].started = d[k].bits_lo = d[k].bits_hi = d[k].rank = d[k].log = 0u;
    d[k].words = 0ull;
    list_at[k] = first_lane(l.lists + 4u * per_dim * min(k, D - 1u));
  }
  double divisor[kMaxDims], inverse[kMaxDims];
#pragma unroll
  for (int k = 0; k < kMaxDims; ++k) {
    divisor[k] = (double)s.P[k];
    inverse[k] = 1.0 / divisor[k];
  }

  // a6: the chunks of a collective that is released join the lists of their
  // first dimensions, in the order of their numbers
  auto add_collective = [&](uint32_t q) {
    for (uint32_t from = 0; from < C; from += 64u) {
      const uint32_t c = from + lane, g = q * C + c;
      const bool exists = c < C;
      const uint32_t st = exists ? state[g] : 0u;
      const uint32_t k0 = (uint32_t)__shfl((int)first_dim, (int)st);
#pragma unroll
      for (uint32_t k = 0; k < (uint32_t)kMaxDims; ++k) {
        const uint64_t m = __builtin_amdgcn_ballot_w64(exists && k0 == k);
        if (k >= D || m == 0ull) continue;
        const uint64_t above = lane < 63u ? m >> (lane + 1u) : 0ull;
        if (exists && k0 == k && above != 0ull) link[g] = (uint16_t)(2u * (g + 1u + (uint32_t)__builtin_ctzll(above)));
        const uint32_t first_lane_of = (uint32_t)__builtin_ctzll(m);
        const uint32_t id = 2u * (q * C + from + first_lane_of);
        const uint32_t last = 2u * (q * C + from + 63u - (uint32_t)__builtin_clzll(m));
        const uint32_t at = lane_get(first_at, first_lane((uint32_t)__shfl((int)st, (int)first_lane_of)));
        const uint32_t to = first_lane((uint32_t)rank_of(q, at));
        const uint32_t word = to >> 6, bit = to & 63u;
        const uint32_t half = lane_get(bit & 32u ? d[k].bits_hi : d[k].bits_lo, word);
        uint32_t* const entry = lists + k * per_dim + to;
        if (half >> (bit & 31u) & 1u) {
          const uint32_t had = first_lane(*entry);
          if (lane == 0u) {
            link[had >> 17] = (uint16_t)id;
            *entry = (had & 0xffffu) | last << 16;
          }
        } else {
          if (lane == 0u) *entry = id | last << 16;
          const uint32_t now_set = half | 1u << (bit & 31u);
          if (bit & 32u) d[k].bits_hi = lane_put(d[k].bits_hi, word, now_set);
          else d[k].bits_lo = lane_put(d[k].bits_lo, word, now_set);
          d[k].words |= 1ull << word;
        }
        __syncthreads();
      }
    }
  };
  TraceWaveRun run;
  const uint32_t stages = gather || rs_only ? D : 2u * D;
  run.now = 0.0;
  run.idle = 15u;
  run.passes = stages * G;
  const uint32_t c_inv = first_lane((uint32_t)((0x80000000ull + C - 1u) / C));
  uint32_t next_release = 0u;
  double rel = has_release ? release[0] : 0.0, now = 0.0, next = nan64();
  for (;;) {
    while (next_release < Q && uniform(rel <= now)) {
      add_collective(first_lane((uint32_t)order[next_release]));
      ++next_release;
      rel = next_release >= Q ? inf64() : has_release ? release[next_release] : 0.0;
    }
    run.now = now;
#pragma unroll
    for (int k = 0; k < kMaxDims; ++k) {   // (scalars, which the compiler does not see here)
      d[k].words = first_lane(d[k].words);
      d[k].running = first_lane(d[k].running);
      d[k].started = first_lane(d[k].started);
    }
    run.idle = first_lane(run.idle);
    run.passes = first_lane(run.passes);
    next = trace_wave_events<kLog, kDivide>(s, t, d, run, rel, c_inv, first_lane(l.records), first_lane(l.record),
                                            first_lane(l.state), list_at, first_lane(gather ? 1u : 0u), divisor, inverse,
                                            (void*)first_lane((uint64_t)rows), first_lane(row_len), first_lane(wide));
    now = lane_get(run.now, 0u);
    if (!uniform(rel < inf64())) break;
    // chunks that arrive at one instant from a release and from a completion
    // would have to be merged by number
    if (uniform(next == rel) || uniform(next < rel)) return WaveOutcome::kNotTaken;
    now = rel;
  }
  r.t_done = now;
  bool empty = true;
#pragma unroll
  for (uint32_t k = 0; k < (uint32_t)kMaxDims; ++k) {
    r.busy[k] = lane_get(d[k].busy, 0u);
    r.executed[k] = d[k].started;
    empty = empty && d[k].words == 0ull;
    // the entries that did not fill the register
    const uint32_t at = (d[k].started & ~63u) + lane;
    if (kLog && at < min(d[k].started, row_len)) {
      if (wide) ((uint16_t*)rows)[k * row_len + at] = (uint16_t)d[k].log;
      else ((uint8_t*)rows)[k * row_len + at] = (uint8_t)d[k].log;
    }
  }
  // every chunk went through, no clock value overflowed and no stage was too
  // short to move the clock (a bound: the shortest one there can be)
  double shortest = inf64();
#pragma unroll
  for (int k = 0; k < kMaxDims; ++k) {
    double x = smallest;
    if (!gather)
      for (int j = 0; j < kMaxDims; ++j) x = j < s.D && j != k ? x / (double)s.P[j] : x;
    if (k < s.D) shortest = min_f64(shortest, s.fix[k] + x * s.coef[k]);
  }
  r.ok = empty && run.idle == 15u && uniform(now < inf64() && now + 0.25 * shortest > now);
  return r.ok ? WaveOutcome::kDone : WaveOutcome::kNotTaken;
}

}  // namespace themis
