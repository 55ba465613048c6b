"""GPU parity of single collectives on each of the two mappings of large batches,
whatever the batch size would choose: one lane per scenario (up to 64 chunks),
and four.  A wavefront holds 16 scenarios in quads, so the edges are 16
scenarios, the chunk capacities, and the scenarios of other NPU counts: of up to
three dimensions in a second turn of their wavefront (with the powers of two
where those are few: 16 in a wavefront of lanes), of four dimensions in the
follow-up kernel, on tables of up to 24 orders and 48 sizes per dimension."""
import numpy as np
import pytest

from test_gpu_mapping import CASES as MAPPING_CASES
from test_gpu_parity import (assert_close, check_batch, gpu, w, _with_collective_types,  # noqa: F401
                             _with_fixed_delay)

pytestmark = pytest.mark.gpu


def _mixed_counts(n, seed, every, dims=None, max_chunks=40):
    """Other NPU counts, and every so many scenarios powers of two."""
    b = w().mixed(n, seed=seed, max_chunks=max_chunks)
    if dims:
        b.ndims[:] = dims
    other = np.arange(n) % every != 0
    b.npus[:, other] = np.random.default_rng(seed).integers(3, 40, (4, int(other.sum())))
    return b


def _large_counts(b, seed):
    """NPU counts over all of their 32 bits (divisions by inverses in the planner)."""
    rng = np.random.default_rng(seed)
    b.npus = np.ascontiguousarray((2 ** rng.uniform(1, 32, b.npus.shape)).astype(np.uint32) | 1)
    return b


CASES = dict(MAPPING_CASES)
CASES.update({
    "1 scenario": lambda W: W.mixed(1, seed=901),
    "17 scenarios": lambda W: W.mixed(17, seed=902, pow2=False),
    "8 of 64 powers of two": lambda W: _mixed_counts(135, 903, 8),
    "32 of 64 powers of two": lambda W: _mixed_counts(135, 904, 2),
    "four dimensions, other counts": lambda W: _mixed_counts(200, 905, 5, dims=4, max_chunks=64),
    "four dimensions, 100 chunks": lambda W: _mixed_counts(70, 906, 3, dims=4, max_chunks=100),
    "three dimensions, 300 chunks": lambda W: _mixed_counts(40, 907, 3, dims=3, max_chunks=300),
    "two of 16 powers of two, four dimensions": lambda W: _mixed_counts(200, 909, 8, dims=4, max_chunks=30),
    "NPU counts of 32 bits": lambda W: _large_counts(_with_collective_types(W.mixed(300, seed=920), 15), 16),
    "types, delays, other counts": lambda W: _with_fixed_delay(_with_collective_types(
        _mixed_counts(300, 908, 3), 13), 14),
})


@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("mapping", ["lane", "quad"])
def test_lanes_and_quads_agree_with_the_oracle(gpu, oracle, mapping, case):
    b = CASES[case](w())
    gpu.themis_set_batch_mapping(gpu.MAPPING_LANE)
    gpu.themis_set_sweep_mapping({"lane": gpu.MAPPING_LANE, "quad": gpu.MAPPING_QUAD}[mapping])
    try:
        check_batch(gpu, oracle, b)
        check_batch(gpu, oracle, b, queue=False, workspace=b.max_chunks > 64)
    finally:
        gpu.themis_set_batch_mapping(gpu.MAPPING_AUTO)
        gpu.themis_set_sweep_mapping(gpu.MAPPING_AUTO)


@pytest.mark.parametrize("max_chunks", [1, 2, 64, 65, 128, 129, 256, 512])
def test_wavefronts_of_one_policy_and_of_both(gpu, oracle, max_chunks):
    """First-in-first-out alone has an event loop of its own: 16 scenarios of it, 16 of
    Smallest-Chunk-First, 16 of either and so on, on powers of two, on other NPU counts
    of up to three dimensions and of four, and with both in a wavefront."""
    for every, dims in ((1, None), (10 ** 9, 3), (10 ** 9, 4), (3, None)):
        b = _with_collective_types(_mixed_counts(131, 980 + max_chunks, every, dims=dims, max_chunks=max_chunks), 20)
        b.chunks[::3] = max_chunks
        kind = np.arange(b.n) // 16 % 3
        b.intra_policy[kind < 2] = kind[kind < 2]
        gpu.themis_set_batch_mapping(gpu.MAPPING_LANE)
        gpu.themis_set_sweep_mapping(gpu.MAPPING_QUAD)
        try:
            check_batch(gpu, oracle, b)
            check_batch(gpu, oracle, b, queue=False)
        finally:
            gpu.themis_set_batch_mapping(gpu.MAPPING_AUTO)
            gpu.themis_set_sweep_mapping(gpu.MAPPING_AUTO)


@pytest.mark.parametrize("n", [15, 17, 511, 512, 513, 1040, 2047])
@pytest.mark.parametrize("max_chunks", [24, 64, 90])
@pytest.mark.parametrize("every", [1, 2, 5, 10 ** 9])
def test_ragged_scenarios_in_turns_of_a_window(gpu, oracle, n, max_chunks, every):
    """512 neighbours are taken by length, 16 at a time; powers of two, and others all or
    every so many (up to three dimensions in the first kernel up to 64 chunks, else in the
    follow-up), with invalid scenarios of every kind among them."""
    b = _mixed_counts(n, 1000 + n, every, max_chunks=max_chunks)
    b = _with_collective_types(b, 21)
    b.bw[0, 3::41] = -1.0
    b.size_bytes[5::43] = np.nan
    b.chunks[7::47] = 0
    b.chunks[9::53] = max_chunks + 1
    b.ndims[11::59] = 5
    for quads in (False, True):
        gpu.themis_set_batch_mapping(gpu.MAPPING_LANE)
        gpu.themis_set_sweep_mapping(gpu.MAPPING_QUAD if quads else gpu.MAPPING_LANE)
        try:
            check_batch(gpu, oracle, b)
            check_batch(gpu, oracle, b, queue=False, workspace=max_chunks > 64)
        finally:
            gpu.themis_set_batch_mapping(gpu.MAPPING_AUTO)
            gpu.themis_set_sweep_mapping(gpu.MAPPING_AUTO)


@pytest.mark.parametrize("n", [1024, 1500, 2047])
@pytest.mark.parametrize("max_chunks", [8, 38, 64])
def test_windows_of_wavefronts_that_differ(gpu, oracle, n, max_chunks):
    """One lane per scenario: in a window of eight wavefronts those with few powers of two
    share turns among each other, and those whose lanes ran, with rows staged in their
    block, take what they have of other counts themselves.  0 to 64 of the 64 scenarios of a
    wavefront are of other counts, up to four dimensions and of three alone, of one length
    and ragged, with invalid ones of every kind."""
    rng = np.random.default_rng(n + max_chunks)
    for ragged, dims in ((True, None), (False, 3), (True, 3)):
        b = w().mixed(n, seed=1300 + n, max_chunks=max_chunks)
        if dims:
            b.ndims[:] = dims
        if not ragged:
            b.chunks[:] = max_chunks
        shares = rng.permutation(np.resize([0, 1, 20, 48, 50, 60, 64, 0], -(-n // 64)))
        for wave, share in enumerate(shares):
            at = 64 * wave + rng.permutation(64)[:share]
            at = at[at < n]
            b.npus[:, at] = rng.integers(3, 40, (4, at.size))
        b = _with_collective_types(b, 23)
        b.bw[0, 3::41] = -1.0
        b.size_bytes[5::43] = np.nan
        b.chunks[7::47] = 0
        b.chunks[9::53] = max_chunks + 1
        b.ndims[11::59] = 5
        gpu.themis_set_batch_mapping(gpu.MAPPING_LANE)
        gpu.themis_set_sweep_mapping(gpu.MAPPING_LANE)
        try:
            check_batch(gpu, oracle, b)
            check_batch(gpu, oracle, b, queue=False, workspace=False)
        finally:
            gpu.themis_set_batch_mapping(gpu.MAPPING_AUTO)
            gpu.themis_set_sweep_mapping(gpu.MAPPING_AUTO)


@pytest.mark.parametrize("max_chunks", [9, 64, 90])
@pytest.mark.parametrize("others", [1, 17, 300, 900])
def test_a_few_scenarios_of_other_counts(gpu, oracle, others, max_chunks):
    """Of 1,100, for the follow-up kernel: those of four dimensions up to 64 chunks, beyond all,
    with scenarios that stall among the powers of two; of one length and ragged."""
    rng = np.random.default_rng(others)
    for ragged in (False, True):
        b = w().mixed(1100, seed=1200 + others, max_chunks=max_chunks)
        if not ragged:
            b.ndims[:] = 4
            b.chunks[:] = max_chunks
        b.npus[:, rng.permutation(b.n)[:others]] = rng.integers(3, 40, (4, others))
        for k in range(4):   # (a stage too short to move the clock)
            b.bw[k, 7 + k::301] = 1e300
        for quads in (False, True):
            gpu.themis_set_batch_mapping(gpu.MAPPING_LANE)
            gpu.themis_set_sweep_mapping(gpu.MAPPING_QUAD if quads else gpu.MAPPING_LANE)
            try:
                check_batch(gpu, oracle, b)
                check_batch(gpu, oracle, b, queue=False, workspace=max_chunks > 64)
            finally:
                gpu.themis_set_batch_mapping(gpu.MAPPING_AUTO)
                gpu.themis_set_sweep_mapping(gpu.MAPPING_AUTO)


@pytest.mark.parametrize("n,chunks", [(16385, 2), (32769, 2), (65536, 2), (65537, 2), (65600, 3), (17000, 70),
                                      (66001, 20), (131073, 1), (131100, 7), (131201, 16), (131300, 17), (131400, 22)])
def test_batch_sizes_around_the_lines(gpu, oracle, n, chunks):
    """Where the mapping changes (from 131,073 scenarios on the lanes' kernels are those
    without a limit of two wavefronts on a SIMD: each layout with rows of whole and of
    odd words, with queue orders and without, with delays), and where the follow-up
    kernel's workgroups look at more scenarios each; all kinds of NPU counts."""
    b = _mixed_counts(n, 910 + chunks, 2, max_chunks=chunks)
    check_batch(gpu, oracle, b, threads=16)
    if n > 65600:
        check_batch(gpu, oracle, b, queue=False, threads=16)
        check_batch(gpu, oracle, _with_fixed_delay(b, 19), threads=16)


@pytest.mark.parametrize("max_chunks,n", [(65, 33), (127, 50), (128, 17), (129, 33), (256, 17), (257, 16)])
def test_sweeps_on_quads_at_the_chunk_capacities(gpu, oracle, max_chunks, n):
    """Every kind of NPU counts at both ends of each capacity, all of its chunks
    used by some scenarios; the last wavefront has empty quads.  (So few wavefronts
    take the layout of 512 chunks where they could take that of 256.)"""
    import torch
    thr = np.array([0.0, 1.0 / 16.0, 0.5])
    gpu.themis_set_sweep_mapping(gpu.MAPPING_QUAD)
    try:
        for delay in (False, True):
            b = _mixed_counts(n, 930 + max_chunks, 2, max_chunks=max_chunks)
            b.chunks[::3] = max_chunks
            if delay:
                b = _with_fixed_delay(b, 17)
            sw = gpu.themis_sweep(gpu.to_device(b), torch.tensor(thr, device="cuda"), 7)
            torch.cuda.synchronize()
            assert_close("sweep", sw.cpu().numpy(), oracle.sweep(b, thr, 7, threads=8))
    finally:
        gpu.themis_set_sweep_mapping(gpu.MAPPING_AUTO)


@pytest.mark.parametrize("max_chunks", [65, 128, 129, 256, 257, 512])
def test_large_sweeps_on_quads_at_the_chunk_capacities(gpu, oracle, max_chunks):
    """More wavefronts than the layout of 512 chunks holds at once, so each capacity runs
    on its own layout, with a list of plans and without one, with delays and without;
    every second network is of other NPU counts."""
    import torch
    n, rng = 5003, np.random.default_rng(960 + max_chunks)
    thr = np.concatenate([[0.0, 0.25], rng.uniform(0, 1, 6)])
    few = np.unique(np.concatenate([[0, n - 1], rng.permutation(n)[:40]]))
    for delay in (False, True):
        b = _mixed_counts(n, 970 + max_chunks, 2, max_chunks=max_chunks)
        b.chunks[::3] = max_chunks
        if delay:
            b = _with_fixed_delay(b, 18)
        want = oracle.sweep(b.take(few), thr, 7, threads=16)
        assert gpu.themis_sweep_scratch_bytes(n, max_chunks, len(thr), 7) > 16
        for scratch in (None, torch.empty(16, dtype=torch.uint8, device="cuda")):   # (16 bytes: no list)
            t = gpu.themis_sweep(gpu.to_device(b), torch.from_numpy(thr).to("cuda"), 7, scratch=scratch)
            torch.cuda.synchronize()
            assert_close("sweep", t.cpu().numpy()[few], want)


@pytest.mark.parametrize("shared", [False, True])
def test_a_sweep_of_more_workgroups_than_one_row_of_the_grid(gpu, oracle, shared):
    """34 million scenarios of up to two chunks under 17 pairs of threshold and scheduler:
    36 million workgroups, in two rows (with a list of plans: the baseline's and one
    per scenario).  The scenarios repeat, so every row of the result has its oracle."""
    import torch
    n, period = 34_000_003, 4096
    b = _mixed_counts(period, 940, 1, max_chunks=2)   # (powers of two)
    b.max_chunks = 65
    thr = np.linspace(0.0, 0.7, 8)
    want = torch.from_numpy(oracle.sweep(b, thr, 7, threads=8)).to("cuda")
    d = gpu.to_device(b)
    at = torch.arange(n, device="cuda") % period
    for f in ("ndims", "size_bytes", "inter_policy", "intra_policy", "threshold", "npus", "bw", "chunks"):
        v = getattr(d, f)
        unsigned = v.dtype == torch.uint32
        v = (v.view(torch.int32) if unsigned else v)[..., at].contiguous()
        setattr(d, f, v.view(torch.uint32) if unsigned else v)
    d.n = n
    scratch = None if shared else torch.empty(16, dtype=torch.uint8, device="cuda")   # (16 bytes: too small for a list)
    t = gpu.themis_sweep(d, torch.from_numpy(thr).to("cuda"), 7, scratch=scratch)
    torch.cuda.synchronize()
    for k in range(0, n, 1024 * period):
        got = t[k:k + 1024 * period]
        exp = want.repeat(-(-got.shape[0] // period), 1, 1)[:got.shape[0]]
        bad = ~torch.isclose(got, exp, rtol=1e-12, atol=0.0, equal_nan=True)
        assert not bool(bad.any()), k + int(bad.nonzero()[0, 0])


@pytest.mark.parametrize("max_chunks", [70, 300])
def test_times_below_the_normal_range_need_no_workspace(gpu, oracle, max_chunks):
    """Beyond 64 chunks on four lanes per scenario: the smallest stage is below the
    normal range, every clock value above zero, and no generic path to fall back on."""
    import torch
    b = w().mixed(100, seed=950, max_chunks=max_chunks)
    b.bw *= 1.5e308 / b.bw.max()
    b.size_bytes *= 1e3 / b.size_bytes.max()
    gpu.themis_set_batch_mapping(gpu.MAPPING_LANE)
    try:
        t = check_batch(gpu, oracle, b, workspace=False)
        assert (t < 1e-299).all() and np.array_equal(t, oracle.simulate_batch(b, oracle.plan_batch(b)[0])[0])
        thr = np.array([0.0, 0.25])
        sw = gpu.themis_sweep(gpu.to_device(b), torch.tensor(thr, device="cuda"), 7)
        torch.cuda.synchronize()
        assert np.array_equal(sw.cpu().numpy(), oracle.sweep(b, thr, 7, threads=8))
    finally:
        gpu.themis_set_batch_mapping(gpu.MAPPING_AUTO)
