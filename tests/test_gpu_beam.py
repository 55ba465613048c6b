"""GPU parity of themis_beam_search_batch with the oracle's beam search
(Sec. 4.1, observation 2: per-chunk orders; the beam keeps `width` partial
schedules where Alg. 1 keeps one).  Times to 1e-12, orders bit for bit: both
sides rank candidates by (time, assignment number) in binary64."""
import math

import numpy as np
import pytest

from test_gpu_parity import assert_close, gpu, w  # noqa: F401

pytestmark = pytest.mark.gpu


def _run(gpu, oracle, b, width, threads=8):
    import torch
    want_t, want_od = oracle.beam_search_batch(b, width, threads=threads)
    got_t, got_od = gpu.themis_beam_search_batch(gpu.to_device(b), width)
    torch.cuda.synchronize()
    got_t, got_od = got_t.cpu().numpy(), got_od.cpu().numpy()
    assert_close("best_t (width %d)" % width, got_t, want_t)
    assert np.array_equal(got_od, want_od)
    return got_t, got_od


def test_beam_search_matches_oracle_on_ragged_batches(gpu, oracle):
    """D 1..4, C 1..12, both queue policies, all collective types, power-of-two
    and other NPU counts (the per-order tables), with and without fixed delays;
    widths 1, 3 and 8."""
    W = w()
    for pow2, seed in ((True, 51), (False, 52)):
        b = W.mixed(160, seed=seed, max_chunks=12, pow2=pow2)
        b.collective_type = (np.arange(b.n) % 3).astype(np.uint8)
        for width in (1, 3, 8):
            t, _ = _run(gpu, oracle, b, width)
            assert np.isfinite(t).sum() >= b.n - 8
        rng = np.random.default_rng(seed)
        b.fixed_delay = np.ascontiguousarray(rng.uniform(0, 5e-6, (4, b.n)))
        _run(gpu, oracle, b, 4)


def test_beam_search_on_tie_rich_networks(gpu, oracle):
    """Dyadic networks: equal times everywhere, so the assignment number decides
    which schedules stay."""
    b = w().dyadic_ties(120, seed=7800, max_chunks=10)
    for width in (1, 2, 6):
        _run(gpu, oracle, b, width)


@pytest.mark.parametrize("width,n,chunks", [(4, 40, 12), (4, 700, 9), (1, 2800, 5), (16, 24, 9), (16, 520, 4),
                                            (5, 1700, 4), (17, 500, 4), (64, 135, 4), (2, 3, 64), (3, 950, 3),
                                            (4, 1023, 3), (4, 1024, 6), (2, 2048, 4), (2, 2049, 3)])
@pytest.mark.parametrize("pow2", [True, False])
def test_beam_widths_around_the_kernel_variants(gpu, oracle, width, n, chunks, pow2):
    """The widths between which the kernel's room changes and batches on both sides
    of the choice between the kernels, with more candidates
    than lanes (ruled out by bounds) and fewer; all collective types, delays,
    networks of four dimensions among the others; sizes whose halvings leave the
    normal range (left to the per-order tables) and whose times single precision
    does not resolve."""
    W, rng = w(), np.random.default_rng(860 + width)
    b = W.mixed(n, seed=861 + width, max_chunks=chunks, pow2=pow2)
    b.chunks[:] = chunks
    b.ndims[::2] = 4
    b.npus[:, ::2] = 2 ** rng.integers(1, 5, (4, (n + 1) // 2)) if pow2 else rng.integers(2, 20, (4, (n + 1) // 2))
    b.bw[:, ::2] = rng.uniform(25e9, 400e9, (4, (n + 1) // 2))
    b.collective_type = (np.arange(n) % 3).astype(np.uint8)
    if n > 3:
        # (bandwidths to match: the shortest stage still moves the clock)
        b.size_bytes = np.where(np.arange(n) % 8 == 5, 3e-307, b.size_bytes)
        b.bw = np.where(np.arange(n) % 8 == 5, b.bw * 1e-20, b.bw)
        b.size_bytes = np.where(np.arange(n) % 8 == 6, 1e-28, b.size_bytes)
    else:
        b.fixed_delay = np.ascontiguousarray(rng.uniform(0, 5e-6, (4, n)))
    t, _ = _run(gpu, oracle, b, width)
    assert np.isfinite(t).sum() >= n // 2


@pytest.mark.parametrize("n", [40, 1100])
@pytest.mark.parametrize("pow2", [True, False])
def test_beam_scenarios_that_no_path_can_simulate(gpu, oracle, n, pow2):
    """A dimension so fast that its stages do not move the clock: no event loop
    takes any schedule of such a scenario, which comes back as NaN / all-ones,
    and the scenarios around it keep their answers."""
    import torch
    W = w()
    b = W.mixed(n, seed=880, max_chunks=6, pow2=pow2)
    b.chunks[:] = np.maximum(b.chunks, 2)
    b.ndims[::5] = 2 + np.arange((n + 4) // 5) % 3
    b.npus[:, ::5] = 4 if pow2 else 3
    b.bw[:, ::5] = 1e11
    b.bw[0, ::5] = 1e300
    want_t, want_od = oracle.beam_search_batch(b, 4, threads=8)
    lost = np.arange(n) % 5 == 0
    assert np.isfinite(want_t[lost]).sum() >= lost.sum() // 2     # (the oracle has an answer)
    want_t[lost], want_od[lost] = np.nan, 0xFF
    got_t, got_od = gpu.themis_beam_search_batch(gpu.to_device(b), 4)
    torch.cuda.synchronize()
    assert_close("best_t", got_t.cpu().numpy(), want_t)
    assert np.array_equal(got_od.cpu().numpy(), want_od)


def test_a_beam_that_drops_nothing_is_the_exhaustive_search(gpu, oracle):
    import torch
    W = w()
    rng = np.random.default_rng(9)
    n = 80
    D = rng.integers(1, 4, n)
    C = np.array([int(rng.integers(1, {1: 7, 2: 7, 3: 3}[int(d)])) for d in D])   # (D!)^C <= 64
    P = [[int(2 ** rng.integers(1, 5)) for _ in range(d)] for d in D]
    bw = [[float(rng.uniform(25e9, 400e9)) for _ in range(d)] for d in D]
    b = W.make_batch(D, P, bw, np.floor(rng.uniform(2 ** 20, 2 ** 30, n)), C, 0,
                     rng.integers(0, 2, n), 0.0, max_chunks=8)
    assert max(math.factorial(int(d)) ** int(c) for d, c in zip(D, C)) <= 64
    d = gpu.to_device(b)
    want_t, want_od = gpu.themis_search_batch(d, 64)
    got_t, got_od = gpu.themis_beam_search_batch(d, 64)
    torch.cuda.synchronize()
    # (the baseline seed cannot win: it is one of the schedules and loses ties)
    assert np.array_equal(got_t.cpu().numpy(), want_t.cpu().numpy())
    assert np.array_equal(got_od.cpu().numpy(), want_od.cpu().numpy())
    _run(gpu, oracle, b, 64)


def test_beam_search_at_64_chunks_is_never_worse_than_the_greedy_plan(gpu, oracle):
    """The paper's default chunk count (Sec. 5.3) on the 4-D bench networks:
    parity on a few scenarios (the oracle takes seconds per scenario), the bound
    by the greedy plan on all."""
    import torch
    W = w()
    b = W.config3(n=6)
    _run(gpu, oracle, b, 2, threads=6)
    big = W.config3(n=512)
    d = gpu.to_device(big)
    t, od = gpu.themis_beam_search_batch(d, 4)
    orders, _ = gpu.themis_plan_batch(d)
    tg, _, _ = gpu.themis_simulate_batch(d, orders, want_queue_order=False)
    tb, _, _ = gpu.themis_simulate_batch(d, od, want_queue_order=False)
    torch.cuda.synchronize()
    t, tg, tb = t.cpu().numpy(), tg.cpu().numpy(), tb.cpu().numpy()
    assert np.isfinite(t).all() and (t <= tg).all()
    assert np.array_equal(t, tb)            # the orders returned reach the time returned


def test_beam_search_refuses_what_it_does_not_cover(gpu):
    import torch
    W = w()
    b = W.mixed(10, seed=3, max_chunks=8)
    d = gpu.to_device(b)
    lib = gpu.lib()
    t = torch.empty(b.n, dtype=torch.float64, device="cuda")
    s = d.c_struct()
    import ctypes as C
    ws = torch.empty(lib.themis_beam_workspace_bytes(b.n, 8, 4), dtype=torch.uint8, device="cuda")
    args = (gpu._ptr(t), None, gpu._ptr(ws), ws.numel(), None)
    assert lib.themis_beam_search_batch(C.byref(s), 0, *args) == -1       # width
    assert lib.themis_beam_search_batch(C.byref(s), 65, *args) == -1
    assert lib.themis_beam_search_batch(C.byref(s), 4, gpu._ptr(t), None, gpu._ptr(ws), 64, None) == -4
    assert lib.themis_beam_workspace_bytes(b.n, 8, 65) == 0
    big = gpu.to_device(W.mixed(4, seed=4, max_chunks=100))
    s2 = big.c_struct()
    assert lib.themis_beam_search_batch(C.byref(s2), 4, *args) == -2      # more than 64 chunk slots
