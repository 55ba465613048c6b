"""GPU parity of the planner and of single collectives' simulation under each
mapping, whatever the batch size would choose: one lane per scenario (beyond 64
chunks four, in the simulation; test_gpu_quads.py has four lanes throughout) and
one wavefront per scenario (whose 64 lanes, 64-entry registers and 512-chunk
LDS arrays put the edges at 64, 65, 128 and 512 chunks).  Smallest and ragged
chunk counts, both policies, all collective types, delays, other NPU counts,
simultaneous completions, values no event loop takes; with and without queue
orders, with fewer scenarios than CUs (evaluated to the end in one kernel) and
more (handed over to the follow-up kernel)."""
import numpy as np
import pytest

from test_gpu_parity import (check_batch, gpu, w, _with_collective_types,  # noqa: F401
                             _with_fixed_delay)

pytestmark = pytest.mark.gpu

CASES = {
    "1 chunk": lambda W: W.mixed(40, seed=801, max_chunks=1, pow2=False),
    "16 chunks": lambda W: W.mixed(300, seed=802, max_chunks=16),
    "63 chunks": lambda W: W.mixed(200, seed=803, max_chunks=63, pow2=False, thr_mode=0),
    "64 chunks": lambda W: W.mixed(400, seed=804, pow2=False),
    "65 chunks": lambda W: W.mixed(120, seed=805, max_chunks=65),
    "128 chunks": lambda W: W.mixed(120, seed=806, max_chunks=128, pow2=False),
    "512 chunks": lambda W: W.mixed(70, seed=807, max_chunks=512, pow2=False),
    "types": lambda W: _with_collective_types(W.mixed(300, seed=808, pow2=False), 8),
    "types, 200 chunks": lambda W: _with_collective_types(W.mixed(90, seed=809, max_chunks=200), 9),
    "delays": lambda W: _with_fixed_delay(_with_collective_types(W.mixed(300, seed=810), 10), 11),
    "ties": lambda W: W.dyadic_ties(300, seed=811),
    "ties, 300 chunks": lambda W: W.dyadic_ties(60, seed=812, max_chunks=300),
    "halvings leave the normal range": lambda W: _tiny(W.mixed(300, seed=813)),
    "the same, few": lambda W: _tiny(W.mixed(60, seed=814, max_chunks=100)),
    "chunks below the normal range": lambda W: _denormal(_with_collective_types(W.mixed(300, seed=816), 12)),
}


def _tiny(b):
    """A third of the sizes where halvings become denormal, a third with one
    bandwidth so large that stages on it do not move the clock."""
    size, bw = b.size_bytes.copy(), b.bw.copy()
    size[::3] = 3e-307
    bw[0, 1::3] = 1e300
    b.size_bytes, b.bw = size, bw
    return b


def _denormal(b):
    """Chunk sizes of 1e-308 and less on bandwidths to match: an All-Gather's grow
    into the normal range, from a size whose exponent field is zero."""
    b.chunks[:] = np.maximum(b.chunks, 32)
    b.size_bytes, b.bw = np.full(b.n, 3e-307), b.bw * 1e-20
    return b


@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("mapping", ["lane", "wave"])
def test_mappings_agree_with_the_oracle(gpu, oracle, mapping, case):
    b = CASES[case](w())
    gpu.themis_set_batch_mapping({"lane": gpu.MAPPING_LANE, "wave": gpu.MAPPING_WAVE}[mapping])
    gpu.themis_set_sweep_mapping({"lane": gpu.MAPPING_LANE, "wave": gpu.MAPPING_AUTO}[mapping])
    try:
        check_batch(gpu, oracle, b)
        check_batch(gpu, oracle, b, queue=False)
        if case == "types":      # a trace's collectives are planned one wavefront each
            check_batch(gpu, oracle, w().config5(n=9, n_coll=5))
    finally:
        gpu.themis_set_batch_mapping(gpu.MAPPING_AUTO)
        gpu.themis_set_sweep_mapping(gpu.MAPPING_AUTO)


@pytest.mark.parametrize("n", [60, 300])
def test_small_sizes_beyond_64_chunks_without_a_workspace(gpu, oracle, n):
    """Halvings below the normal range are for the per-order tables, which need no
    workspace: the answer is there on both sides of the number of CUs, up to
    which one kernel does everything."""
    b = w().mixed(n, seed=815, max_chunks=100)
    b.chunks[:] = 100
    tiny = np.arange(n) % 3 == 0
    b.size_bytes = np.where(tiny, 3e-307, b.size_bytes)
    b.bw = np.where(tiny, b.bw * 1e-20, b.bw)      # (the shortest stage still moves the clock)
    for queue in (True, False):
        t = check_batch(gpu, oracle, b, queue=queue, workspace=False)
        assert np.isfinite(t[tiny]).all()


@pytest.mark.parametrize("n", [1, 256, 257, 2048, 2049, 3072, 3073, 4096, 4097])
def test_batch_sizes_around_the_choice_of_the_mapping(gpu, oracle, n):
    """Both kinds of NPU counts (from 2,049 to 3,072 scenarios each kind is planned
    on its own mapping); invalid scenarios; one or two chunks."""
    b = w().mixed(n, seed=820, max_chunks=9, pow2=False)
    b.npus[:, ::2] = 1 << np.floor(np.log2(b.npus[:, ::2])).astype(np.int64)
    b.size_bytes[n // 2::97] = 0.0 if n > 1 else b.size_bytes[0]
    check_batch(gpu, oracle, b)
    check_batch(gpu, oracle, w().mixed(n, seed=821, max_chunks=2, pow2=False))


def test_trace_collectives_planned_on_both_mappings(gpu, oracle):
    """2,255 collectives of which some scenarios have fewer than others."""
    b = w().config5(n=205, n_coll=11)
    b.npus[:, ::2] = [[6], [12], [24], [2]]
    b.n_coll = (1 + np.arange(b.n) % 11).astype(np.uint32)
    b.size_bytes = b.size_bytes.copy()
    b.intra_policy[::3] = 0
    check_batch(gpu, oracle, b)


@pytest.mark.parametrize("bound,n,chunks,dims", [(1, 7, 1, 1), (64, 40, 6, 2), (65, 40, 6, 2), (576, 30, 2, 4),
                                                 (1296, 3, 4, 3), (1296, 7000, 4, 3), (13824, 9, 3, 4)])
@pytest.mark.parametrize("pow2", [True, False])
def test_searches_with_one_and_with_several_wavefronts_per_scenario(gpu, oracle, bound, n, chunks, dims, pow2):
    """themis_search_batch where a wavefront simulates all of its assignments
    at once, where it rules most of them out by their bounds, and where several
    share a scenario; collective types and delays among them."""
    import torch
    from test_gpu_parity import assert_close
    W, rng = w(), np.random.default_rng(830 + bound + n)
    P = [[int(2 ** rng.integers(1, 5)) if pow2 else int(rng.integers(2, 20)) for _ in range(dims)]
         for _ in range(n)]
    b = W.make_batch([dims] * n, P, rng.uniform(25e9, 400e9, (n, dims)).tolist(),
                     np.floor(rng.uniform(2 ** 20, 2 ** 30, n)), rng.integers(max(1, chunks - 1), chunks + 1, n),
                     1, rng.integers(0, 2, n), 0.0, max_chunks=chunks)
    b = _with_fixed_delay(_with_collective_types(b, 1), 2)
    d = gpu.to_device(b)
    got_t, got_o = gpu.themis_search_batch(d, bound)
    torch.cuda.synchronize()
    few = np.arange(n) if n < 100 else rng.permutation(n)[:100]
    want_t, want_o = oracle.search_batch(b.take(few), bound, threads=8)
    assert_close("best_t", got_t.cpu().numpy()[few], want_t)
    assert np.array_equal(got_o.cpu().numpy()[few], want_o)


@pytest.mark.parametrize("bound,n,chunks,dims", [(1, 3300, 64, 1), (1, 5000, 1, 1), (2, 3073, 1, 2), (16, 3500, 4, 2),
                                                 (24, 3333, 1, 4), (32, 26000, 5, 2), (30, 3100, 5, 2), (6, 3201, 17, 3)])
def test_tiny_searches_of_many_scenarios(gpu, oracle, bound, n, chunks, dims):
    """A lane per assignment and several scenarios to a wavefront (64 of one
    assignment, ten of six, two of 24 or 30), those of other NPU counts among
    them, each with fewer assignments than the bound or more, which is no answer;
    invalid scenarios and sizes below the normal range; in batches whose last
    wavefronts are not full."""
    import torch
    from test_gpu_parity import assert_close
    W, rng = w(), np.random.default_rng(890 + bound + n)
    P = np.where(rng.random((n, 1)) < 0.6, 2 ** rng.integers(1, 5, (n, dims)), rng.integers(2, 20, (n, dims)))
    size = np.floor(rng.uniform(2 ** 20, 2 ** 30, n))
    size[7::31] = 0.0
    size[11::37] = 3e-307
    bw = rng.uniform(25e9, 400e9, (n, dims))
    bw[11::37] *= 1e-20
    most = chunks if dims < 3 or chunks == 1 else 2      # (36 assignments: beyond the bound)
    b = W.make_batch([dims] * n, P.tolist(), bw.tolist(), size, rng.integers(1, most + 1, n), 1,
                     rng.integers(0, 2, n), 0.0, max_chunks=chunks)
    b = _with_collective_types(b, 1)
    few = np.unique(np.concatenate([np.arange(140), np.arange(n - 70, n), rng.permutation(n)[:200]]))
    delayed = b.take(np.arange(n))
    delayed.size_bytes[11::37] = 2.0 ** 20    # (beside a delay the tiny stages would not move the clock)
    for batch in (b, _with_fixed_delay(delayed, 2)):
        got_t, got_o = gpu.themis_search_batch(gpu.to_device(batch), bound)
        torch.cuda.synchronize()
        want_t, want_o = oracle.search_batch(batch.take(few), bound, threads=8)
        assert_close("best_t", got_t.cpu().numpy()[few], want_t)
        assert np.array_equal(got_o.cpu().numpy()[few], want_o)
        assert np.isfinite(want_t).sum() > len(few) // 4


def test_searches_whose_times_single_precision_does_not_resolve(gpu, oracle):
    """The bounds that rule assignments out are in single precision: times of
    1e-45 .. 1e-37 seconds are denormal there."""
    import torch
    from test_gpu_parity import assert_close
    W, rng, n = w(), np.random.default_rng(850), 60
    b = W.make_batch([3] * n, rng.integers(2, 20, (n, 3)).tolist(), rng.uniform(25e9, 400e9, (n, 3)).tolist(),
                     10.0 ** rng.uniform(-35, -26, n), [3] * n, 1, rng.integers(0, 2, n), 0.0, max_chunks=3)
    got_t, got_o = gpu.themis_search_batch(gpu.to_device(b), 216)
    torch.cuda.synchronize()
    want_t, want_o = oracle.search_batch(b, 216, threads=8)
    assert_close("best_t", got_t.cpu().numpy(), want_t)
    assert np.array_equal(got_o.cpu().numpy(), want_o)


@pytest.mark.parametrize("n,max_chunks,n_thr,mask,per_scenario,pow2",
                         [(16001, 9, 8, 7, False, True), (15000, 20, 5, 6, True, False),
                          (9000, 64, 32, 7, False, True), (5003, 70, 8, 7, False, True),
                          (2700, 257, 8, 5, False, True), (6000, 3, 8, 2, True, True),
                          (17003, 2, 8, 7, True, False), (16385, 2, 8, 7, False, True),
                          (100, 64, 8, 7, False, False), (3, 512, 8, 7, True, True)])
def test_sweeps_whose_thresholds_share_plans(gpu, oracle, n, max_chunks, n_thr, mask, per_scenario, pow2):
    """themis_sweep where it looks for thresholds that give the same plan (from
    a few thousand wavefronts on), on both mappings, with thresholds that are
    not valid and scenarios that go to the follow-up passes; and where it takes
    a wavefront per evaluation."""
    import torch
    from test_gpu_parity import assert_close
    W, rng = w(), np.random.default_rng(840 + n)
    b = W.mixed(n, seed=841 + n, max_chunks=max_chunks, pow2=pow2)
    b.size_bytes = np.where(np.arange(n) % 50 == 7, 3e-307, b.size_bytes)   # denormal halvings
    b.size_bytes[5 % n] = 0.0 if n > 100 else b.size_bytes[5 % n]           # an invalid scenario
    thr = np.concatenate([[0.0, 0.25, np.nan, 0.25], rng.uniform(0, 1, n_thr - 4)])
    if per_scenario:
        thr = np.ascontiguousarray(rng.permuted(np.repeat(thr[:, None], n, axis=1), axis=0))
    d = gpu.to_device(b)
    ws = gpu.alloc_workspace(gpu.themis_workspace_bytes(n * n_thr * 3, max_chunks)) if max_chunks > 64 else None
    out = torch.full((n, n_thr, bin(mask).count("1")), -1.0, dtype=torch.float64, device="cuda")
    gpu.themis_sweep(d, torch.from_numpy(thr).cuda(), mask, thr_per_scenario=per_scenario, t_done=out,
                     workspace=ws)
    torch.cuda.synchronize()
    few = np.unique(np.concatenate([[5 % n, 7 % n], rng.permutation(n)[:80]]))
    keep = np.ascontiguousarray(thr[:, few]) if per_scenario else thr
    want = oracle.sweep(b.take(few), keep, mask, thr_per_scenario=per_scenario, threads=8)
    assert_close("sweep", out.cpu().numpy()[few], want)


@pytest.mark.parametrize("chunks", [1, 15, 16, 31, 32, 33, 63, 64, 65, 127, 128, 512])
@pytest.mark.parametrize("mapping", ["wave", "quad", "lane"])
def test_turns_under_smallest_chunk_first(gpu, oracle, mapping, chunks):
    """A chunk's last Reduce-Scatter and first All-Gather are one stage on wavefronts and
    quads: two records of a log that leaves 64 at a time, two operations in the counts; with
    sizes at the end of the normal range, where equal ones would have to wait for each other."""
    from test_gpu_parity import _with_fixed_delay
    b = w().mixed(72, seed=1100 + chunks, max_chunks=chunks, pow2=False)
    b.ndims[:] = 1 + np.arange(b.n) % 4
    b.npus[:, ::3] = 2 ** (1 + np.arange(4 * 24).reshape(4, 24) % 5)
    b.chunks[:] = chunks
    b.intra_policy[:] = np.arange(b.n) % 5 != 0
    b.size_bytes[6::17] = 2.3e-308 * chunks * 2.0 ** np.arange(b.n)[6::17]
    gpu.themis_set_batch_mapping({"wave": gpu.MAPPING_WAVE}.get(mapping, gpu.MAPPING_LANE))
    gpu.themis_set_sweep_mapping({"quad": gpu.MAPPING_QUAD, "lane": gpu.MAPPING_LANE}.get(mapping, gpu.MAPPING_AUTO))
    try:
        check_batch(gpu, oracle, b)
        check_batch(gpu, oracle, _with_fixed_delay(b, 22), queue=False)
    finally:
        gpu.themis_set_batch_mapping(gpu.MAPPING_AUTO)
        gpu.themis_set_sweep_mapping(gpu.MAPPING_AUTO)


def test_a_sweep_whose_scratch_does_not_fit_goes_without(gpu, monkeypatch):
    """The list of plans is an extra: a caller whose batch leaves no room for it
    gets the same results, and one that keeps it around hands it in."""
    import torch
    n = 30000
    d = gpu.to_device(w().mixed(n, seed=871, max_chunks=64))
    thr = torch.linspace(0.0, 0.5, 8, dtype=torch.float64, device="cuda")
    need = gpu.themis_sweep_scratch_bytes(n, 64, 8, 7)
    assert need > 0
    own = gpu.themis_sweep(d, thr, 7)
    given = gpu.themis_sweep(d, thr, 7, scratch=torch.empty(need, dtype=torch.uint8, device="cuda"))

    def no_room(*args, **kwargs):
        raise torch.OutOfMemoryError("no room")
    monkeypatch.setattr(gpu, "alloc_workspace", no_room)
    without = gpu.themis_sweep(d, thr, 7)
    torch.cuda.synchronize()
    bits = [t.view(torch.int64).cpu() for t in (own, given, without)]
    assert torch.equal(bits[0], bits[1]) and torch.equal(bits[0], bits[2])


@pytest.mark.parametrize("n", [9, 7000])
def test_search_of_a_workspace_that_holds_marks(gpu, oracle, n):
    """Every 64th scenario is left to the per-order tables (halvings below the
    normal range), some are not valid, and the caller's workspace happens to hold
    the bits with which the first kernel marks what it leaves: only rows that it
    has written may be taken for marked ones."""
    import torch
    from test_gpu_parity import assert_close
    W, rng, C, bound = w(), np.random.default_rng(870), 3, 216
    P = rng.integers(2, 20, (n, 3))
    size = np.floor(rng.uniform(2 ** 20, 2 ** 30, n))
    size[5::7] = 0.0
    size[::64] = 1e-308 * C * P[::64].prod(axis=1)
    b = W.make_batch([3] * n, P.tolist(), rng.uniform(25e9, 400e9, (n, 3)).tolist(), size, C, 1,
                     rng.integers(0, 2, n), 0.0, max_chunks=C)
    mark = 0x7ff8a5a55a5a0001
    ws = torch.full((gpu.themis_search_workspace_bytes(n, bound) // 8,), mark, dtype=torch.int64, device="cuda")
    got_t, got_o = gpu.themis_search_batch(gpu.to_device(b), bound, ws)
    torch.cuda.synchronize()
    few = np.arange(n) if n < 100 else np.unique(np.concatenate([np.arange(0, n, 64), rng.permutation(n)[:60]]))
    want_t, want_o = oracle.search_batch(b.take(few), bound, threads=8)
    assert_close("best_t", got_t.cpu().numpy()[few], want_t)
    assert np.array_equal(got_o.cpu().numpy()[few], want_o)
    # (the first words of a row hold what the wavefronts of a scenario found)
    rows = ws.view(n, bound).cpu().numpy()[:, 2 * -(-bound // 64):]
    kept = (rows == mark).all(axis=1)
    left = np.arange(n) % 64 == 0
    assert kept[~left].all() and not kept[left].any()
