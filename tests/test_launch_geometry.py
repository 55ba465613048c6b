"""How the entry points lay out their launches, without a GPU: in a process of its
own the library's hipLaunchKernel is one that writes down kernel, grid and
workgroup, and refuses what HIP refuses (2^32 threads or more along one direction
of a grid, more LDS than a workgroup can have).  The batches exist as sizes only:
the host never looks at their arrays."""
import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RECORDER = r"""
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
typedef struct { uint32_t x, y, z; } dim3_t;
int hipLaunchKernel(const void* f, dim3_t g, dim3_t b, void** args, size_t lds, void* stream) {
  Dl_info at;
  const int refused = (uint64_t)g.x * b.x >> 32 || (uint64_t)g.y * b.y >> 32 || g.y > 65535u || lds > 163840u ||
                      !g.x || !g.y || !g.z;
  (void)args; (void)stream;
  printf("%s %u %u %u %u %d\n", dladdr(f, &at) && at.dli_sname ? at.dli_sname : "?", g.x, g.y, g.z, b.x, refused);
  fflush(stdout);
  return refused ? 9 : 0;   /* hipErrorInvalidConfiguration */
}
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int what, int d) { (void)what; (void)d; *v = atoi(getenv("RECORDED_CUS")); return 0; }
"""

CALLER = r"""
import ctypes, json, sys
ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
from paper_2110_04478_amd import binding
L = binding.lib()
fake = 0x10000
for name, n, max_chunks, extra in json.loads(sys.argv[2]):
    b = binding._Batch()
    b.n, b.max_chunks, b.threshold_mode = n, max_chunks, 1
    for f in ("ndims", "npus", "bw", "size_bytes", "chunks", "inter_policy", "intra_policy", "threshold"):
        setattr(b, f, fake)
    L.themis_set_batch_mapping(extra.get("batch_mapping", 0))
    L.themis_set_sweep_mapping(extra.get("sweep_mapping", 0))
    if "max_coll" in extra:
        b.max_coll, b.n_coll, b.coll_size = extra["max_coll"], fake, fake
    ref, big = ctypes.byref(b), 1 << 62
    print("call", flush=True)
    if name == "simulate":
        st = L.themis_simulate_batch(ref, fake, fake, fake, fake, fake, big, None)
    elif name == "plan":
        st = L.themis_plan_batch(ref, fake, None, None)
    else:
        st = L.themis_sweep_with_scratch(ref, extra["n_thr"], fake, 0, extra["mask"], fake, fake, big,
                                         fake, big if extra.get("scratch") else 0, None)
    print("status", st, flush=True)
"""


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    """launches([(entry point, n, max_chunks, {..}), ..]) -> [(status, [(kernel, workgroups, rows, refused), ..]), ..]"""
    from paper_2110_04478_amd.csrc.build import ensure_built
    ensure_built()
    d = tmp_path_factory.mktemp("recorder")
    (d / "r.c").write_text(RECORDER)
    (d / "call.py").write_text(CALLER)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", str(d / "r.so"), str(d / "r.c"), "-ldl"], check=True)

    def run(calls, cus=256):
        env = dict(os.environ, RECORDED_CUS=str(cus), PYTHONPATH=ROOT)
        out = subprocess.run([sys.executable, str(d / "call.py"), str(d / "r.so"), json.dumps(calls)],
                             env=env, check=True, capture_output=True, text=True).stdout
        results = []
        for line in out.splitlines():
            w = line.split()
            if line == "call":
                results.append([None, []])
            elif w[0] == "status":
                results[-1][0] = int(w[1])
            else:
                x, y, z, _, refused = map(int, w[1:])
                results[-1][1].append((w[0], x * y * z, y, bool(refused)))
        assert len(results) == len(calls)
        return results

    return run


def _blocks(result, kernel):
    found = [l for l in result[1] if kernel in l[0]]
    assert len(found) >= 1, (kernel, result)
    return found


def test_batches_of_hundreds_of_millions_are_launched(launches):
    """Four lanes per scenario beyond 64 chunks: what one lane each took (fewer than
    2^32 threads: 252 million scenarios of a sweep under 17 pairs, 2^32 of a
    simulation) is launched, with a workgroup for every 16."""
    calls = [("sweep", n, c, dict(n_thr=8, mask=mask, scratch=scratch))
             for n in (63_161_280, 63_161_290, 70_000_000, 252_000_000) for c in (65, 128, 256, 512)
             for mask in (6, 7) for scratch in (False, True)]
    calls += [("sweep", 17, 65, dict(n_thr=(1 << 26) - 1, mask=2))]   # (67 million thresholds)
    calls += [("simulate", n, c, {}) for n in ((1 << 30) - 16, 1 << 30, (1 << 32) - 1) for c in (65, 512)]
    for (name, n, c, extra), got in zip(calls, launches(calls)):
        assert got[0] == 0 and not any(l[3] for l in got[1]), (name, n, c, extra, got)
        workgroups, rows = _blocks(got, "quad_kernel")[0][1:3]
        need = -(-n // 16)
        if name == "sweep":
            n_pol = bin(extra["mask"]).count("1")
            roles = extra["n_thr"] * n_pol - (extra["n_thr"] - 1 if extra["mask"] & 1 else 0)
            need = need * roles
            if any("sweep_plans" in l[0] for l in got[1]):   # (the baseline's and as many as there can be jobs)
                need = (-(-n // 16) if extra["mask"] & 1 else 0) + -(-n * 8 // 16) * 2
        assert need <= workgroups < need + (1 << 25) and (rows == 1) == (need <= 1 << 25), (name, n, c, extra, got)


def test_traces_of_large_batches_are_launched(launches):
    """Four lanes per trace take 2^30 and more (single chunks); a wavefront per trace
    is not asked for where a launch has no room for them, whatever the mapping."""
    calls = [("simulate", n, 1, dict(max_coll=1, batch_mapping=m)) for n in (1 << 30, (1 << 32) - 64) for m in (0, 1, 3)]
    calls += [("plan", 1 << 26, 1, dict(batch_mapping=3)), ("simulate", 1 << 26, 1, dict(batch_mapping=3))]
    for call, got in zip(calls, launches(calls)):
        assert got[0] == 0 and not any(l[3] for l in got[1]), (call, got)


def test_a_grid_that_block_numbers_do_not_reach_is_an_error(launches):
    got = launches([("simulate", (1 << 36) + 16, 65, {})])[0]
    assert got[0] != 0


@pytest.mark.parametrize("cus", [256, 64, 20])
def test_four_lanes_per_scenario_until_one_each_fill_the_gpu(launches, cus):
    """Up to 64 chunks the line between the two is a wavefront of lanes on every SIMD,
    whatever part of the GPU the device is (below 4,097 scenarios, a wavefront each)."""
    line = 256 * cus
    quads, lanes = launches([("simulate", line, 64, {}), ("simulate", line + 1, 64, {})], cus=cus)
    assert any("simulate_quad_kernel" in l[0] for l in quads[1])
    assert not any("simulate_quad_kernel" in l[0] for l in lanes[1]) and any("simulate_kernel" in l[0] for l in lanes[1])


@pytest.mark.parametrize("cus", [256, 48])
def test_batches_of_two_wavefronts_per_simd(launches, cus):
    """Up to two wavefronts of lanes for every SIMD the simulation has registers for no
    third one there, and the planner takes four wavefronts for a group of 64."""
    line = 512 * cus
    for chunks in (9, 64):
        for n, few in ((line - 100, True), (line, True), (line + 1, False)):
            plan, sim = launches([("plan", n, chunks, {}), ("simulate", n, chunks, {})], cus=cus)
            assert plan[1][0][1] == -(-n // 64) * (4 if few else 1), (n, chunks, plan)
            kernel = _blocks(sim, "simulate_kernel")[0]
            assert ("TwoPerSimd" in kernel[0]) == few and kernel[1] == -(-n // 64), (n, chunks, sim)
