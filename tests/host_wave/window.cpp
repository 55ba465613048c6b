// The order of a window's scenarios (themis_window.hpp), on the CPU.
//   window <largest length there can be> in out
// in: 512 lengths (u32, 0: not among them).  out: turn by turn the scenario of each quad
// (u32, all-ones: none), until the last turn.
//   window turns <n> out
// out: window, turn and turns of the window of every workgroup of a batch of n (u32).
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

int main(int, char** argv) {
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
