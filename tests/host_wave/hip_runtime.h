// A wavefront on the CPU: what the headers of the event loops need of HIP, for g++.
// The 64 lanes are coroutines that run one after the other and meet at every
// instruction that exchanges values between lanes, so the program is the device's
// own, statement by statement (inline assembly has been taken out of the copy that is
// compiled here: see test_quads_on_host.py).  LDS blocks and workspaces end where
// memory that cannot be touched begins.
#pragma once
#include <math.h>
#include <signal.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>
#include <ucontext.h>
#include <unistd.h>

#define __device__
#define __host__
#define __forceinline__ inline __attribute__((always_inline))

struct uint4 { uint32_t x, y, z, w; };
struct dim3_host { uint32_t x, y, z; };
static dim3_host threadIdx;
static inline uint32_t min(uint32_t a, uint32_t b) { return a < b ? a : b; }
static inline uint32_t max(uint32_t a, uint32_t b) { return a > b ? a : b; }

static inline uint64_t f64_bits(double v) { uint64_t b; memcpy(&b, &v, 8); return b; }
static inline double f64_of(uint64_t b) { double v; memcpy(&v, &b, 8); return v; }
static inline double __longlong_as_double(long long b) { return f64_of((uint64_t)b); }
static inline long long __double_as_longlong(double v) { return (long long)f64_bits(v); }
static inline int __double2hiint(double v) { return (int)(f64_bits(v) >> 32); }
static inline int __double2loint(double v) { return (int)f64_bits(v); }
static inline double __hiloint2double(int hi, int lo) { return f64_of((uint64_t)(uint32_t)hi << 32 | (uint32_t)lo); }
static inline int __clz(int v) { return v ? __builtin_clz((uint32_t)v) : 32; }
static inline uint32_t __umulhi(uint32_t a, uint32_t b) { return (uint32_t)((uint64_t)a * b >> 32); }
static inline uint32_t __umul24(uint32_t a, uint32_t b) { return (a & 0xffffffu) * (b & 0xffffffu); }

// -- lanes ----------------------------------------------------------------------------
struct Wave {
  ucontext_t scheduler, lane[64];
  bool done[64];
  uint32_t met[64];
  uint64_t value[2][64];
  uint32_t kind[2][64];
  uint32_t now;
  void (*body)(void*);
  void* arg;
};
static Wave wave;
// All lanes give a value and see everybody's; kind: they have to be at the same one.
static inline const uint64_t* meet(uint64_t v, uint32_t kind) {
  const uint32_t me = wave.now, n = wave.met[me]++;
  wave.value[n & 1u][me] = v;
  wave.kind[n & 1u][me] = kind;
  swapcontext(&wave.lane[me], &wave.scheduler);
  for (uint32_t l = 0; l < 64u; ++l)
    if (wave.met[l] <= n || wave.kind[n & 1u][l] != kind) {
      printf("lanes %u and %u do not meet\n", me, l);
      exit(4);
    }
  return wave.value[n & 1u];
}
static void lane_main() {
  wave.body(wave.arg);
  wave.done[wave.now] = true;
  swapcontext(&wave.lane[wave.now], &wave.scheduler);
}
static void run_wave(void (*body)(void*), void* arg) {
  static char* stacks = (char*)malloc(64u << 18);
  wave.body = body;
  wave.arg = arg;
  for (uint32_t l = 0; l < 64u; ++l) {
    getcontext(&wave.lane[l]);
    wave.lane[l].uc_stack.ss_sp = stacks + ((size_t)l << 18);
    wave.lane[l].uc_stack.ss_size = 1u << 18;
    wave.done[l] = false;
    wave.met[l] = 0;
    makecontext(&wave.lane[l], lane_main, 0);
  }
  for (bool left = true; left;) {
    left = false;
    for (uint32_t l = 0; l < 64u; ++l) {
      if (wave.done[l]) continue;
      wave.now = l;
      threadIdx.x = l;
      swapcontext(&wave.scheduler, &wave.lane[l]);
      left = true;
    }
  }
}
static inline uint32_t me() { return wave.now; }
#define __syncthreads() ((void)meet(0, 1))
#define __threadfence_block() ((void)0)
#define __builtin_amdgcn_fence(order, scope) ((void)0)
#define __builtin_amdgcn_wave_barrier() ((void)meet(0, 2))
static inline uint64_t __builtin_amdgcn_ballot_w64(bool p) {
  const uint64_t* v = meet(p, 3);
  uint64_t m = 0;
  for (uint32_t l = 0; l < 64u; ++l) m |= v[l] << l;
  return m;
}
static inline int __builtin_amdgcn_readfirstlane(int x) { return (int)meet((uint32_t)x, 4)[0]; }
static inline int __builtin_amdgcn_mov_dpp(int x, int perm, int, int, bool) {
  const uint32_t l = me();
  return (int)meet((uint32_t)x, 5u + (uint32_t)perm)[(l & ~3u) | ((uint32_t)perm >> (2u * (l & 3u)) & 3u)];
}
static inline int __shfl_xor(int x, int off) {
  const uint32_t l = me();
  return (int)meet((uint32_t)x, 0x1000u)[l ^ (uint32_t)off];
}
static inline int __shfl_up(int x, uint32_t off) {
  const uint32_t l = me();
  return (int)meet((uint32_t)x, 0x1001u)[l < off ? l : l - off];
}
static inline int __builtin_amdgcn_readlane(int x, int l) { return (int)meet((uint32_t)x, 0x1002u)[l]; }
static inline uint32_t __builtin_amdgcn_mbcnt_lo(uint32_t m, uint32_t n) {
  return n + (uint32_t)__builtin_popcount(me() < 32u ? m & ((1u << me()) - 1u) : m);
}
static inline uint32_t __builtin_amdgcn_mbcnt_hi(uint32_t m, uint32_t n) {
  return n + (uint32_t)(me() < 32u ? 0 : __builtin_popcount(m & ((1u << (me() - 32u)) - 1u)));
}
static inline uint32_t __builtin_amdgcn_udot4(uint32_t a, uint32_t b, uint32_t c, bool) {
  for (int j = 0; j < 32; j += 8) c += (a >> j & 0xffu) * (b >> j & 0xffu);
  return c;
}
static inline int __builtin_amdgcn_sdot4(int a, int b, int c, bool) {
  for (int j = 0; j < 32; j += 8) c += (int8_t)((uint32_t)a >> j) * (int8_t)((uint32_t)b >> j);
  return c;
}
static inline uint32_t __builtin_amdgcn_alignbit(uint32_t hi, uint32_t lo, uint32_t by) {
  return (uint32_t)(((uint64_t)hi << 32 | lo) >> (by & 31u));
}
static inline uint32_t __builtin_amdgcn_perm(uint32_t hi, uint32_t lo, uint32_t which) {
  uint32_t r = 0;
  for (int j = 0; j < 32; j += 8) {
    const uint32_t b = which >> j & 0xffu;
    if (b > 7u) { printf("perm\n"); exit(4); }
    r |= (uint32_t)(((uint64_t)hi << 32 | lo) >> (8u * b) & 0xffu) << j;
  }
  return r;
}
// (not run here)
typedef int __amdgpu_buffer_rsrc_t;
static inline int __builtin_amdgcn_make_buffer_rsrc(void*, int, long, int) { abort(); }
static inline void __builtin_amdgcn_raw_buffer_store_b8(uint8_t, int, uint32_t, int, int) { abort(); }
static inline bool __builtin_amdgcn_inverse_ballot_w64(uint64_t) { abort(); }

// -- memory that ends where it ends ---------------------------------------------------
struct Guarded { uint8_t *reserve, *block; size_t bytes; };
static Guarded guarded[2];
static constexpr size_t kGuard = (size_t)1 << 36;
static void outside(int, siginfo_t* info, void*) {
  for (const Guarded& g : guarded)
    if ((uint8_t*)info->si_addr >= g.reserve && (uint8_t*)info->si_addr < g.reserve + 2u * kGuard)
      printf("lane %u is at byte %ld of a block of %zu\n", wave.now, (long)((uint8_t*)info->si_addr - g.block), g.bytes);
  printf("outside\n");
  fflush(stdout);
  _exit(3);
}
// A block of that many bytes, of old contents; at_end: its end is the border (else its start).
static uint8_t* guard(uint32_t which, size_t bytes, bool at_end) {
  Guarded& g = guarded[which];
  if (!g.reserve) {
    g.reserve = (uint8_t*)mmap(nullptr, 2u * kGuard, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    struct sigaction a = {};
    a.sa_sigaction = outside;
    a.sa_flags = SA_SIGINFO;
    sigaction(SIGSEGV, &a, nullptr);
    sigaction(SIGBUS, &a, nullptr);
  }
  const size_t pages = (bytes + 4095u) & ~(size_t)4095u;
  uint8_t* const middle = g.reserve + kGuard;
  mmap(middle - (64u << 20), 128u << 20, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE | MAP_FIXED, -1, 0);
  if (mprotect(middle, pages, PROT_READ | PROT_WRITE) != 0) abort();
  memset(middle, 0xa5, pages);
  g.block = at_end ? middle + (pages - bytes) : middle;
  g.bytes = bytes;
  return g.block;
}
