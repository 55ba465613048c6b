"""GPU parity of traces under each mapping, whatever the batch size would choose:
one lane per trace, four (a quad: what is released together on powers of two,
sixteen traces to a wavefront, four dimensions in a launch of their own), and one
wavefront per trace, whose edges are 64
chunks of a collective, 64 operations of a dimension (the queue orders leave a
register then, as bytes up to 127 chunk slots), 64 size ranks (a word of the
bitmap) and 4,096 (its end), and the LDS of a launch, which has enough for up to
three dimensions of powers of two in the first one."""
import numpy as np
import pytest

from test_gpu_quads import _large_counts
from test_gpu_parity import (_add_trace, _with_collective_types, _with_fixed_delay, assert_close,  # noqa: F401
                             check_batch, gpu, mapping, w, widen_queue)

pytestmark = pytest.mark.gpu


def _trace(n, seed, max_chunks, max_coll, pow2=True, equal_sizes=False, dims=None, full=False, ties=False):
    rng = np.random.default_rng(seed)
    b = w().dyadic_ties(n, seed=seed, max_chunks=max_chunks) if ties else \
        w().mixed(n, seed=seed, max_chunks=max_chunks, pow2=pow2)
    b = _add_trace(b, rng, max_coll, pow2_sizes=equal_sizes)
    if dims:
        b.ndims[:] = dims
    if full:
        b.n_coll[:], b.chunks[:] = max_coll, max_chunks
    return b


def _released(b, seed, step=0.0):
    rng = np.random.default_rng(seed)
    b.release_time = np.ascontiguousarray(rng.integers(0, 4, b.coll_size.shape) * step if step else
                                          rng.uniform(0, 1, b.coll_size.shape) ** 3 * 5e-3)
    return b


def _bottleneck(b):
    """One dimension so slow that hundreds of chunks wait for it, on lists they share
    and on many others."""
    b.bw[1] *= 0.02
    return b


def _fifo(b):
    b.intra_policy[:] = 0
    return b


CASES = {
    "one chunk": lambda: _trace(90, 1, 1, 70),
    "127 slots": lambda: _trace(40, 2, 127, 1, full=True),
    "128 slots": lambda: _trace(40, 3, 32, 4, full=True),
    "63 chunks": lambda: _trace(30, 4, 63, 3),
    "65 chunks": lambda: _trace(30, 5, 65, 5, pow2=False),
    "512 chunks": lambda: _trace(6, 6, 512, 3, full=True),
    "256 collectives, 4-D": lambda: _trace(9, 7, 3, 256, dims=4, full=True),
    "256 collectives, equal sizes": lambda: _trace(9, 8, 3, 256, equal_sizes=True, full=True),
    "80 and 90 collectives, 4-D, other counts": lambda: _trace(7, 9, 3, 90, pow2=False, dims=4),
    "other counts, releases": lambda: _released(_trace(90, 10, 17, 8, pow2=False), 1),
    "types, delays, releases": lambda: _released(_with_fixed_delay(_with_collective_types(
        _trace(120, 11, 16, 9), 2), 3), 4),
    "NPU counts of 32 bits": lambda: _large_counts(_trace(60, 19, 9, 5), 9),
    "types, other counts": lambda: _with_collective_types(_trace(120, 12, 9, 7, pow2=False), 5),
    "1 trace": lambda: _trace(1, 15, 20, 12, dims=3),
    "17 traces, long queues": lambda: _bottleneck(_trace(17, 16, 30, 40, dims=3)),
    "four dimensions, delays": lambda: _with_fixed_delay(_bottleneck(_trace(40, 17, 21, 20, dims=4)), 8),
    "first-in-first-out": lambda: _fifo(_trace(60, 18, 33, 11)),
    "ties": lambda: _trace(150, 13, 16, 6, equal_sizes=True, ties=True),
    "ties, releases": lambda: _released(_trace(150, 14, 16, 6, equal_sizes=True, ties=True), 6, step=2.0 ** -12),
}


@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("lanes", ["lane", "quad", "wave"])
def test_traces_agree_with_the_oracle(gpu, oracle, lanes, case):
    b = CASES[case]()
    gpu.themis_set_batch_mapping(gpu.MAPPING_WAVE if lanes == "wave" else gpu.MAPPING_LANE)
    gpu.themis_set_sweep_mapping(gpu.MAPPING_QUAD if lanes == "quad" else gpu.MAPPING_LANE)
    try:
        t = check_batch(gpu, oracle, b)
        assert np.isfinite(t).all()
        check_batch(gpu, oracle, b, queue=False)
    finally:
        gpu.themis_set_batch_mapping(gpu.MAPPING_AUTO)
        gpu.themis_set_sweep_mapping(gpu.MAPPING_AUTO)


@pytest.mark.parametrize("released", [True, False])
def test_invalid_traces(gpu, oracle, mapping, released):
    """Bad sizes, counts of collectives and networks, malformed order codes: NaN and
    all-ones, with valid traces beside them in their wavefront; stages that do not move
    the clock and sizes that leave the normal range go on to the other paths.
    (Four lanes per trace take what is released together.)"""
    import torch
    b = _trace(64, 21, 9, 5)
    if released:
        b = _released(b, 7)
    b.coll_size[0, ::8], b.npus[0, 2::8] = 0.0, 1
    b.n_coll[3::8], b.n_coll[4::8] = 0, 6
    b.coll_size[:, 5::8] = 3e-307
    b.bw[0, 6::8] = 1e300
    t = check_batch(gpu, oracle, b)
    good = np.flatnonzero(np.isfinite(t))
    assert len(good) >= 24
    orders = oracle.plan_batch(b)[0].reshape(b.n, b.max_coll, b.max_chunks)
    bad = good[::3]
    for j, i in enumerate(bad):   # (of the first chunk, of some, of the last)
        q, c = [(0, 0), (b.n_coll[i] // 2, b.chunks[i] // 2), (b.n_coll[i] - 1, b.chunks[i] - 1)][j % 3]
        orders[i, q, c] = 0xff if j % 2 else (1 if b.ndims[i] == 1 else 0)
    orders = np.ascontiguousarray(orders.reshape(b.n, -1))
    want_t, want_qo, want_busy = oracle.simulate_batch(b, orders)
    assert np.isnan(want_t[bad]).all()
    d = gpu.to_device(b)
    ws = gpu.alloc_workspace(gpu.themis_workspace_bytes(d.n, d.max_chunks, d.max_coll))
    t, qo, busy = gpu.themis_simulate_batch(d, torch.from_numpy(orders).cuda(), workspace=ws)
    torch.cuda.synchronize()
    assert_close("t_done", t.cpu().numpy(), want_t)
    assert np.array_equal(widen_queue(qo), want_qo)
    assert_close("busy", busy.cpu().numpy(), want_busy)
