"""GPU parity of the planner and of single collectives' simulation under each
lane mapping, whatever the batch size would choose: one lane per scenario and
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
}


def _tiny(b):
    """A third of the sizes where halvings become denormal, a third with one
    bandwidth so large that stages on it do not move the clock."""
    size, bw = b.size_bytes.copy(), b.bw.copy()
    size[::3] = 3e-307
    bw[0, 1::3] = 1e300
    b.size_bytes, b.bw = size, bw
    return b


@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("mapping", ["lane", "wave"])
def test_mappings_agree_with_the_oracle(gpu, oracle, mapping, case):
    b = CASES[case](w())
    gpu.themis_set_batch_mapping({"lane": gpu.MAPPING_LANE, "wave": gpu.MAPPING_WAVE}[mapping])
    try:
        check_batch(gpu, oracle, b)
        check_batch(gpu, oracle, b, queue=False)
        if case == "types":      # a trace's collectives are planned one wavefront each
            check_batch(gpu, oracle, w().config5(n=9, n_coll=5))
    finally:
        gpu.themis_set_batch_mapping(gpu.MAPPING_AUTO)


@pytest.mark.parametrize("n", [1, 256, 257, 3073, 4096, 4097])
def test_batch_sizes_around_the_choice_of_the_mapping(gpu, oracle, n):
    check_batch(gpu, oracle, w().mixed(n, seed=820, max_chunks=9, pow2=False))
