// The order of a window's scenarios (themis_window.hpp), on the CPU.
//   window <largest length there can be> in out
// in: 512 lengths (u32, 0: not among them).  out: turn by turn the scenario of each quad
// (u32, all-ones: none), until the last turn.
//   window turns <n> out
// out: window, turn and turns of the window of every workgroup of a batch of n (u32).
//   window marked <n> <max_chunks> <4: of four dimensions, 3: the others; o, p: first those of other
//     NPU counts, powers of two> in out
// in: ndims (u8), npus (u32, 4 rows), chunks (u32), 1 where a scenario is marked (u8), n of
// each.  out: for each turn of the first window that has marks its number and its 16 scenarios
// (u32, all-ones: none).
#include <vector>
#include "themis_window.hpp"

using namespace themis;

static uint32_t lengths[kWindow], turns, most;
static uint32_t chosen[kWindowTurns][16];
static uint8_t* lds;

static void order(void*) {
  uint32_t own[kWindowGroups];
  for (uint32_t g = 0; g < kWindowGroups; ++g) own[g] = lengths[64u * g + threadIdx.x];
  const QuadWindow w(most, lds, own);
  for (uint32_t turn = 0; turn < w.turns(); ++turn) {
    uint32_t which;
    const bool exists = w.take(turn, lds, which);
    chosen[turn][threadIdx.x >> 2] = exists ? which : ~0u;
  }
  turns = w.turns();
}

static themis_batch_t batch;
static std::vector<uint8_t> is_marked;
static std::vector<uint32_t> found;
static bool four;
static LeftFirst first;
static void marked(void*) {
  uint32_t own = 0u;
  for (uint32_t g = 0; g < kWindowGroups; ++g)
    if (64u * g + threadIdx.x < batch.n && is_marked[64u * g + threadIdx.x]) own |= 1u << g;
  MarkedWindow w(batch, 0u, four);
  if (!w.any(own)) return;
  uint32_t turns;
  const QuadWindow order = w.order(batch, 0u, first, own, lds, turns);
  for (; turns != 0u; turns &= turns - 1u) {
    const uint32_t turn = (uint32_t)__builtin_ctz(turns);
    uint32_t which;
    const bool exists = order.take(turn, lds, which);
    if (threadIdx.x == 0u) found.push_back(turn);
    if ((threadIdx.x & 3u) == 0u) found.push_back(exists ? which : ~0u);
  }
}
template <typename T>
static const T* take(FILE* f, size_t n) {
  T* v = (T*)malloc(n * sizeof(T));
  if (fread(v, sizeof(T), n, f) != n) exit(5);
  return v;
}

int main(int, char** argv) {
  if (strcmp(argv[1], "marked") == 0) {
    batch.n = (uint64_t)atoll(argv[2]);
    batch.max_chunks = (uint32_t)atoi(argv[3]);
    four = argv[4][0] == '4';
    first = argv[4][1] == 'p' ? LeftFirst::kPow2 : argv[4][1] == 'o' ? LeftFirst::kOthers : LeftFirst::kAll;
    FILE* f = fopen(argv[5], "rb");
    batch.ndims = take<uint8_t>(f, batch.n);
    batch.npus = take<uint32_t>(f, 4u * batch.n);
    batch.chunks = take<uint32_t>(f, batch.n);
    const uint8_t* m = take<uint8_t>(f, batch.n);
    is_marked.assign(m, m + batch.n);
    lds = guard(0u, 1056u, true);
    run_wave(marked, nullptr);
    f = fopen(argv[6], "wb");
    fwrite(found.data(), 4u, found.size(), f);
    fclose(f);
    printf("ran\n");
    return 0;
  }
  if (strcmp(argv[1], "turns") == 0) {
    const uint64_t n = (uint64_t)atoll(argv[2]);
    FILE* out = fopen(argv[3], "wb");
    for (uint32_t block = 0; block * 16ull < n; ++block) {
      const WindowTurn t = window_turn(n, block);
      const uint32_t v[3] = {(uint32_t)t.window, t.turn, t.turns};
      fwrite(v, sizeof v, 1, out);
    }
    fclose(out);
    printf("ran\n");
    return 0;
  }
  most = (uint32_t)atoi(argv[1]);
  FILE* f = fopen(argv[2], "rb");
  if (!f || fread(lengths, sizeof lengths, 1, f) != 1) return 5;
  lds = guard(0u, 1056u, true);
  run_wave(order, nullptr);
  f = fopen(argv[3], "wb");
  fwrite(chosen, sizeof chosen[0], turns, f);
  fclose(f);
  printf("ran\n");
  return 0;
}
