// The event loops with four lanes per scenario and per trace, on the CPU.
//   queues single <chunk capacity> <0: powers of two, 3 or 4: tables of that many dimensions> <n> <max_chunks> in out
//   queues trace <dimensions> <n> <max_chunks> <max_coll> in out
// in: the arrays of a batch one after the other, then the order codes (a wavefront has empty
// quads between the others).  out: per scenario t_done and busy (f64), taken (u32), then its
// queue orders (u16).
#include <vector>
#include "themis_generic.hpp"
#include "themis_trace_quad.hpp"

using namespace themis;

struct Input {
  themis_batch_t b{};
  std::vector<std::vector<uint8_t>> keep;
  FILE* f;
  template <typename T>
  T* take(size_t n) {
    keep.emplace_back(n * sizeof(T));
    if (n && fread(keep.back().data(), sizeof(T), n, f) != n) abort();
    return (T*)keep.back().data();
  }
};
static Input in;
static const uint8_t* orders;
static bool at_end;
struct Out { double t, busy[4]; uint32_t taken; };
static std::vector<Out> results;
static std::vector<uint16_t> entries;
static uint8_t *lds, *area;

// the scenario of the lane's quad in this wavefront (its quads are not all in use)
static uint32_t wave_number;
static const uint32_t kUsed = 11u;   // quads of a wavefront with a scenario
static bool scenario_of_quad(uint64_t& i) {
  const uint32_t quad = threadIdx.x >> 2;
  const bool used = quad % 3u != 1u;
  i = (uint64_t)wave_number * kUsed + quad - (quad + 1u) / 3u;
  const bool exists = used && i < in.b.n;
  if (!exists) i = 0;
  return exists;
}

static void store(bool exists, uint64_t i, bool taken, double t, double busy) {
  if (!exists) return;
  Out& o = results[i];
  o.busy[threadIdx.x & 3u] = busy;
  if ((threadIdx.x & 3u) == 0u) { o.t = t; o.taken = taken; }
}

template <typename L, uint32_t kDims>
static void single(void*) {
  uint64_t i;
  const bool exists = scenario_of_quad(i);
  const uint32_t k = threadIdx.x & 3u;
  const Scenario s = load_scenario(in.b, i);
  const uint32_t D = (uint32_t)s.D;
  const double chunk = in.b.size_bytes[i] / (double)s.C;
  const bool scf = in.b.intra_policy[i] == THEMIS_INTRA_SCF;
  const uint8_t* const row = orders + i * in.b.max_chunks;
  uint16_t* const put_at = entries.data() + (i * 4u + k) * 2u * in.b.max_chunks;
  auto put = [&](uint32_t e, uint32_t entry) { put_at[e] = (uint16_t)entry; };
  QuadQueue<L> queue(lds);
  QuadResult r;
  if constexpr (kDims == 0u) {
    FastScenario fs;
    const bool runs = fast_eligible(s, chunk, L::kCap, fs) && exists;
    for (uint32_t c = 0; runs && c < s.C; ++c)
      if ((row[c] & 3u) == k)
        queue.add(c | ((quad_row(D) + quad_order(stored_code(s, fs, row[c]), D)) & 31u) << 9 | (fs.gather ? 1u << L::kPhaseBit : 0u));
    const Pow2Model pow2(s, fs, scf);
    r = simulate_quad<L, true>(QuadPow2<L, true>(s, pow2, k, lds), queue,
                               (uint32_t)(pow2.ranktab >> (4u * (fs.state0 & 15u))) & 15u,
                               runs ? (pow2.one_phase() ? D : 2u * D) * s.C : 0u, pow2.t_min(D), put);
  } else {
    using Table = QuadTable<L, kDims>;
    const bool gather = s.ctype == THEMIS_COLL_ALL_GATHER;
    uint32_t used = 0u;
    auto order_of = [&](uint32_t code) { return quad_order(gather ? reverse_code(code, s.D) : code, D) % Table::kOrders; };
    for (uint32_t c = 0; exists && c < s.C; ++c) used |= 1u << order_of(row[c]);
    const Table model(s, chunk, scf, used, lds);
    for (uint32_t c = 0; exists && c < s.C; ++c)
      if ((row[c] & 3u) == k) queue.add(c | Table::state_of(order_of(row[c]), gather ? 1u : 0u) << 9);
    r = simulate_quad<L, true>(model, queue, model.cls0,
                               exists ? (s.ctype == THEMIS_COLL_ALL_REDUCE ? 2u * D : D) * s.C : 0u, model.t_min, put);
  }
  store(exists, i, r.ok, r.t_done, r.busy);
}

static uint32_t trace_dims;
static uint32_t trace_stride;
static void trace(void*) {
  uint64_t i;
  const bool exists = scenario_of_quad(i);
  const themis_batch_t& b = in.b;
  const Scenario s = load_scenario(b, i);
  const uint32_t Q = b.n_coll[i], slots = b.max_chunks * b.max_coll, k = threadIdx.x & 3u;
  FastScenario fs;
  double smallest = inf64();
  bool takes = exists && s.valid && (uint32_t)s.D <= trace_dims;
  for (uint32_t q = 0; q < Q; ++q) {
    const double chunk = b.coll_size[(size_t)q * b.n + i] / (double)s.C;
    takes = takes && fast_eligible(s, chunk, THEMIS_MAX_CHUNKS, fs);
    smallest = min_f64(smallest, chunk);
  }
  fast_eligible(s, s.valid ? b.coll_size[i] / (double)s.C : 1.0, THEMIS_MAX_CHUNKS, fs);
  const TraceQuadLayout l = trace_quad_layout(slots, trace_dims, b.max_coll);
  const uint8_t* const row = orders + i * slots;
  uint16_t* const put_at = entries.data() + (i * 4u + k) * 2u * slots;
  const TraceQuadResult r = simulate_trace_quad<true>(
      s, fs, takes ? Q : 0u, b.intra_policy[i] == THEMIS_INTRA_SCF, smallest, l, lds, area, trace_stride,
      [&](uint32_t q, uint32_t c) {
        uint32_t v = 0u;
        for (uint32_t j = 0; j < 4u && c + j < s.C; ++j) v |= (uint32_t)row[(size_t)q * b.max_chunks + c + j] << (8u * j);
        return v;
      },
      [&](uint32_t q) { return b.coll_size[(size_t)q * b.n + i] / (double)s.C; },
      [&](uint32_t e, uint32_t entry) { put_at[e] = (uint16_t)entry; });
  store(exists, i, takes && r.ok, r.t_done, r.busy);
}

template <typename L, uint32_t kDims>
static size_t single_bytes() {
  if constexpr (kDims == 0u) return QuadPow2<L, true>::kBytes;
  else return QuadTable<L, kDims>::kBytes;
}
struct Kind { void (*body)(void*); size_t bytes; };
template <uint32_t kCap>
static Kind kind_of(uint32_t dims) {
  using L = LayoutQuad<kCap, 16>;
  using L3 = LayoutQuad<kCap, 12u, 3u>;
  using L4 = LayoutQuad<kCap, 48u>;
  return dims == 0u ? Kind{single<L, 0u>, single_bytes<L, 0u>()}
       : dims == 3u ? Kind{single<L3, 3u>, single_bytes<L3, 3u>()} : Kind{single<L4, 4u>, single_bytes<L4, 4u>()};
}

int main(int argc, char** argv) {
  const bool is_trace = strcmp(argv[1], "trace") == 0;
  themis_batch_t& b = in.b;
  b.n = (uint64_t)atoll(argv[is_trace ? 3 : 4]);
  b.max_chunks = (uint32_t)atoi(argv[is_trace ? 4 : 5]);
  b.max_coll = is_trace ? (uint32_t)atoi(argv[5]) : 0u;
  in.f = fopen(argv[argc - 2], "rb");
  b.ndims = in.take<uint8_t>(b.n);
  b.npus = in.take<uint32_t>(4u * b.n);
  b.bw = in.take<double>(4u * b.n);
  b.size_bytes = in.take<double>(b.n);
  b.chunks = in.take<uint32_t>(b.n);
  b.intra_policy = in.take<uint8_t>(b.n);
  b.fixed_delay = in.take<double>(4u * b.n);
  b.collective_type = in.take<uint8_t>(b.n);
  if (is_trace) {
    b.n_coll = in.take<uint32_t>(b.n);
    b.coll_size = in.take<double>((size_t)b.max_coll * b.n);
  }
  const size_t slots = (size_t)b.max_chunks * (is_trace ? b.max_coll : 1u);
  orders = in.take<uint8_t>(b.n * slots);
  results.resize(b.n);
  entries.assign(b.n * 4u * 2u * slots, 0xffffu);
  Kind kind;
  if (is_trace) {
    trace_dims = (uint32_t)atoi(argv[2]);
    trace_stride = trace_layout(b.max_chunks, b.max_coll).bytes;
    const TraceQuadLayout l = trace_quad_layout((uint32_t)slots, trace_dims, b.max_coll);
    if (l.region > trace_stride) { printf("region\n"); return 5; }
    kind = Kind{trace, l.lds};
  } else {
    const uint32_t cap = (uint32_t)atoi(argv[2]), dims = (uint32_t)atoi(argv[3]);
    kind = cap == 64u ? kind_of<64>(dims) : cap == 128u ? kind_of<128>(dims)
         : cap == 256u ? kind_of<256>(dims) : kind_of<512>(dims);
  }
  for (wave_number = 0; (uint64_t)wave_number * kUsed < b.n; ++wave_number)
    for (int side = 0; side < 2; ++side) {   // (the border behind the block, and before it)
      lds = guard(0u, kind.bytes, side == 0);
      if (is_trace) area = guard(1u, 16u * (size_t)trace_stride, side == 0);
      run_wave(kind.body, nullptr);
    }
  FILE* out = fopen(argv[argc - 1], "wb");
  for (uint64_t i = 0; i < b.n; ++i) {
    fwrite(&results[i].t, 8, 1, out);
    fwrite(results[i].busy, 8, 4, out);
    fwrite(&results[i].taken, 4, 1, out);
  }
  fwrite(entries.data(), 2, entries.size(), out);
  fclose(out);
  printf("ran\n");
  return 0;
}
