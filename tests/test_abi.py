"""The C ABI library builds, loads and exports every symbol the header
declares (no compute calls: runs without a GPU)."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module", autouse=True)
def built_library():
    """hipcc cross-compiles without a GPU; compiles only when no library is in the tree."""
    from paper_2110_04478_amd.csrc.build import ensure_built
    ensure_built()


def declared_functions():
    text = open(os.path.join(ROOT, "include", "themis.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(themis_[a-z_]+)\s*\(", text)))


def test_header_declares_the_three_entry_points():
    names = declared_functions()
    for must in ("themis_plan_batch", "themis_simulate_batch", "themis_sweep"):
        assert must in names


def test_library_exports_every_declared_symbol():
    from paper_2110_04478_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2110_04478_amd.csrc import build
        build.build()
    L = ctypes.CDLL(binding.LIB_PATH)
    for name in declared_functions():
        assert hasattr(L, name), f"{name} is declared in themis.h but not exported"


def test_host_side_helpers():
    from paper_2110_04478_amd import binding
    L = binding.lib()
    assert binding.themis_version() >= 100
    assert L.themis_status_string(0) == b"success"
    assert L.themis_status_string(-1) and L.themis_status_string(-99)
    assert binding.themis_queue_entry_bytes(64) == 1
    assert binding.themis_queue_entry_bytes(127) == 1
    assert binding.themis_queue_entry_bytes(128) == 2
    assert binding.themis_queue_entry_bytes(64, 200) == 2
    assert binding.themis_workspace_bytes(0, 64) == 0
    assert binding.themis_workspace_bytes(1000, 64) >= 1000 * 64 * 8


def test_sweep_scratch_is_only_asked_for_where_it_can_be_used():
    """The list of plans is built by a power of two of lanes per scenario, in a
    grid of less than 2^32 lanes, and counted in 32 bits."""
    from paper_2110_04478_amd import binding
    need = binding.lib().themis_sweep_scratch_bytes
    assert need(65536, 64, 8, 7) > 0 and need(100_000_000, 64, 17, 7) > 0
    assert need(200_000_000, 64, 17, 7) == 0      # 32 lanes each
    assert need(1 << 28, 64, 16, 6) == 0          # 2^32 plans
    assert need(65536, 64, 3, 7) == 0 and need(65536, 64, 33, 7) == 0 and need(16, 64, 8, 7) == 0


def test_argument_errors_are_reported_without_a_device():
    """NULL / out-of-range arguments are rejected on the host before any HIP
    call, so this needs no GPU."""
    from paper_2110_04478_amd import binding
    L = binding.lib()
    assert L.themis_plan_batch(None, None, None, None) == -1
    b = binding._Batch()
    b.n, b.max_chunks, b.threshold_mode = 4, 0, 0
    assert L.themis_plan_batch(ctypes.byref(b), None, None, None) == -1
    b.max_chunks = 1024
    assert L.themis_plan_batch(ctypes.byref(b), None, None, None) == -1
    b.max_chunks, b.threshold_mode = 64, 7
    assert L.themis_simulate_batch(ctypes.byref(b), None, None, None, None, None, 0, None) == -1
    b.threshold_mode = 0
    assert L.themis_plan_batch(ctypes.byref(b), None, None, None) == -1   # NULL arrays
    b.n = 0
    assert L.themis_plan_batch(ctypes.byref(b), None, None, None) == 0    # empty batch: no-op
    assert L.themis_sweep(ctypes.byref(b), 0, None, 0, 7, None, None, 0, None) == -1


def test_misaligned_workspace_is_rejected_on_the_host():
    """The workspace must be 16-byte aligned; the check comes before any HIP
    call (the pointers below are never dereferenced on the host)."""
    from paper_2110_04478_amd import binding
    L = binding.lib()
    b = binding._Batch()
    b.n, b.max_chunks, b.threshold_mode = 4, 64, 0
    fake = 0x10000
    for f in ("ndims", "npus", "bw", "size_bytes", "chunks", "inter_policy", "intra_policy",
              "threshold"):
        setattr(b, f, fake)
    assert L.themis_simulate_batch(ctypes.byref(b), fake, fake, None, None, fake + 8, 1 << 20,
                                   None) == -4
    assert L.themis_sweep(ctypes.byref(b), 1, fake, 0, 7, fake, fake + 4, 1 << 20, None) == -4
    assert L.themis_search_batch(ctypes.byref(b), 16, fake, None, fake + 4, 1 << 20, None) == -4


def test_no_lane_crossing_instruction_right_after_an_exec_switch():
    """The inline-assembly blocks that make each dimension's lanes the active
    ones in turn are opaque to the compiler's hazard recogniser: no instruction
    that reads other lanes may follow the last exec write within the wait
    states the target asks for (checked on the compiled device code)."""
    from paper_2110_04478_amd.csrc import build
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc here")
    blocks, found = build.exec_hazards(build.device_assembly())
    assert blocks > 0          # the blocks are there (else this test checks nothing)
    assert not found, found
