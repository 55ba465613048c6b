"""The event loops with four lanes per scenario and per trace, run on the CPU: the
headers' own code, a wavefront as 64 coroutines (tests/host_wave), against the oracle.
LDS block and workspace are bordered by memory that cannot be touched, and shifts by
more than a word has bits, first bits of zero and divisions by zero end the program:
no lane may read outside of its layout, also where a quad has no scenario, where
nothing ends in it and where nothing waits."""
import os
import re
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2110_04478_amd", "csrc")
HEADERS = ("themis_device.hpp", "themis_fast.hpp", "themis_ring.hpp", "themis_quad.hpp", "themis_generic.hpp", "themis_trace.hpp",
           "themis_trace_quad.hpp", "themis_window.hpp")
INSTEAD = {"v_min_f64": "r = fmin(a, b);", "v_max_f64": "r = fmax(a, b);", "": ""}


def _without_assembly(text):
    """Each asm statement becomes what it stands for, or an abort()."""
    out, at = [], 0
    for m in re.finditer(r"\basm\b\s*(?:volatile)?\s*\(", text):
        if m.start() < at:
            continue
        depth, end = 1, m.end()
        while depth:
            depth += {"(": 1, ")": -1}.get(text[end], 0)
            end += 1
        first = re.match(r'\s*"(\w*)', text[m.end():])
        out += [text[at:m.start()], INSTEAD.get(first.group(1) if first else None, "abort();")]
        at = text.index(";", end) + 1
    return "".join(out) + text[at:]


def _headers(d):
    """The headers as g++ takes them."""
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(open(os.path.join(HERE, "host_wave", "hip_runtime.h")).read())
    for h in HEADERS:
        (d / h).write_text(_without_assembly(open(os.path.join(CSRC, h)).read()))
    return d


def _program(tmp_path_factory, name):
    d = _headers(tmp_path_factory.mktemp("host_wave"))
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-w", "-fsanitize=shift-exponent,builtin,integer-divide-by-zero",
                    "-fsanitize-undefined-trap-on-error", "-I", str(d), "-I", os.path.join(HERE, "..", "include"),
                    "-o", str(d / name), os.path.join(HERE, "host_wave", name + ".cpp")], check=True)
    return d


@pytest.fixture(scope="module")
def queues(tmp_path_factory):
    d = _program(tmp_path_factory, "queues")

    def run(b, orders, *kind):
        """-> (t_done, busy [4, n], taken, queue orders) of the batch."""
        n, trace = b.n, b.n_coll is not None
        with open(d / "in", "wb") as f:
            for a, dt in ((b.ndims, np.uint8), (b.npus, np.uint32), (b.bw, np.float64), (b.size_bytes, np.float64),
                          (b.chunks, np.uint32), (b.intra_policy, np.uint8),
                          (np.zeros((4, n)) if b.fixed_delay is None else b.fixed_delay, np.float64),
                          (np.zeros(n) if b.collective_type is None else b.collective_type, np.uint8)):
                f.write(np.ascontiguousarray(a, dtype=dt).tobytes())
            if trace:
                f.write(np.ascontiguousarray(b.n_coll, dtype=np.uint32).tobytes())
                f.write(np.ascontiguousarray(b.coll_size, dtype=np.float64).tobytes())
            f.write(np.ascontiguousarray(orders, dtype=np.uint8).tobytes())
        sizes = [n, b.max_chunks] + ([b.max_coll] if trace else [])
        p = subprocess.run([str(d / "queues"), "trace" if trace else "single", *map(str, kind), *map(str, sizes),
                            str(d / "in"), str(d / "out")], capture_output=True, text=True, timeout=300)
        assert p.returncode == 0 and p.stdout == "ran\n", (p.returncode, p.stdout[-500:])
        raw = open(d / "out", "rb").read()
        rows = np.frombuffer(raw, dtype=np.dtype([("t", "<f8"), ("busy", "<f8", 4), ("taken", "<u4")]), count=n)
        entries = np.frombuffer(raw, dtype="<u2", offset=rows.nbytes).reshape(n, 4, -1)
        return rows["t"], rows["busy"].T, rows["taken"], entries

    return run


def _mixed(n, seed, max_chunks, dims=None, pow2=True, delays=True):
    from paper_2110_04478_amd import workloads
    rng = np.random.default_rng(seed)
    b = workloads.mixed(n, seed=seed, max_chunks=max_chunks, pow2=pow2)
    if dims:
        b.ndims = np.minimum(b.ndims, dims) if dims < 4 else np.full(n, 4, np.uint8)
    b.collective_type = rng.integers(0, 3, n).astype(np.uint8)
    if delays:
        b.fixed_delay = np.ascontiguousarray(rng.uniform(0, 2e-6, (4, n)))
    return b


def _ties(n, seed, max_chunks):
    from paper_2110_04478_amd import workloads
    return workloads.dyadic_ties(n, seed=seed, max_chunks=max_chunks)


def _any_orders(b, seed):
    """Permutations that no planner makes."""
    rng = np.random.default_rng(seed)
    orders = np.full((b.n, b.max_chunks), 0xff, np.uint8)
    for i in range(b.n):
        for c in range(int(b.chunks[i])):
            p = rng.permutation(int(b.ndims[i]))
            orders[i, c] = sum(int(k) << (2 * j) for j, k in enumerate(p))
    return orders


def _check(oracle, queues, b, orders, *kind):
    t, busy, taken, entries = queues(b, orders, *kind)
    want_t, want_entries, want_busy = oracle.simulate_batch(b, orders)
    assert taken.all() and np.array_equal(t, want_t)
    for k in range(4):
        assert np.array_equal(np.where(k < b.ndims, busy[k], 0.0), np.where(k < b.ndims, want_busy[k], 0.0))
    assert np.array_equal(entries, want_entries)


@pytest.mark.parametrize("cap,chunks,n", [(64, 2, 30), (64, 9, 30), (64, 64, 11), (128, 128, 11), (256, 200, 11), (512, 300, 11)])
@pytest.mark.parametrize("kind", ["powers of two", "ties", "any orders", "tables"])
def test_single_collectives(oracle, queues, cap, chunks, n, kind):
    if kind == "tables":   # every NPU count, ties among them, up to three dimensions and four
        for dims in (3, 4):
            b = _mixed(n, 40 + cap, chunks, dims=dims, pow2=False)
            _check(oracle, queues, b, _any_orders(b, cap), cap, dims)
            b = _ties(n, 60 + cap, chunks)
            b.ndims = np.minimum(b.ndims, dims)
            _check(oracle, queues, b, _any_orders(b, 7), cap, dims)
        return
    b = _ties(n, 20 + cap, chunks) if kind == "ties" else _mixed(n, 30 + cap, chunks)
    orders = _any_orders(b, cap) if kind == "any orders" else oracle.plan_batch(b)[0]
    _check(oracle, queues, b, orders, cap, 0)


@pytest.mark.parametrize("cap,chunks,n", [(64, 1, 14), (64, 64, 11), (128, 127, 11), (256, 256, 11), (512, 512, 11)])
@pytest.mark.parametrize("dims", [0, 3, 4])
def test_first_in_first_out_alone(oracle, queues, cap, chunks, n, dims):
    """The event loop of wavefronts without Smallest-Chunk-First (dims: tables of that
    many dimensions, 0: powers of two), every instant a tie, and none."""
    for b in (_ties(n, 140 + cap, chunks), _mixed(n, 150 + cap, chunks, dims=dims or None, pow2=not dims)):
        if dims:
            b.ndims = np.minimum(b.ndims, dims)
        b.intra_policy[:] = 0
        _check(oracle, queues, b, _any_orders(b, cap), cap, dims)


@pytest.mark.parametrize("max_chunks,max_coll,dims,n", [(1, 1, 3, 14), (5, 1, 4, 14), (9, 6, 3, 14), (16, 20, 4, 11), (8, 40, 3, 11)])
def test_traces(oracle, queues, max_chunks, max_coll, dims, n):
    rng = np.random.default_rng(max_coll)
    for ties in (False, True):
        b = _ties(n, 80 + max_coll, max_chunks) if ties else _mixed(n, 90 + max_coll, max_chunks, dims=dims)
        b.ndims = np.minimum(b.ndims, dims)
        b.max_coll = max_coll
        b.n_coll = rng.integers(1, max_coll + 1, n).astype(np.uint32)
        b.coll_size = 2.0 ** rng.integers(16, 22, (max_coll, n)) if ties else rng.uniform(1e5, 1e9, (max_coll, n))
        b.release_time = None
        _check(oracle, queues, b, oracle.plan_batch(b)[0], dims)


def _short_times(n, max_chunks, dims):
    """Stage times below the smallest normal number, sizes above it."""
    b = _mixed(n, 120 + dims, max_chunks, dims=dims, delays=False)
    b.bw = b.bw * (1.5e308 / b.bw.max())
    b.size_bytes = b.size_bytes * (1e3 / b.size_bytes.max())
    return b


@pytest.mark.parametrize("dims", [3, 4])
def test_times_below_the_normal_range(oracle, queues, dims):
    """A scaled product rounds twice there: the loop for powers of two leaves such
    scenarios, the one on tables (the model's own operations) takes them."""
    b = _short_times(22, 90, dims)
    orders = oracle.plan_batch(b)[0]
    want = oracle.simulate_batch(b, orders)[0]
    assert (want < 1e-299).all() and (want > 0).all()
    t, _, taken, _ = queues(b, orders, 128, 0)
    assert (taken == 0).sum() > b.n // 2 and np.array_equal(t[taken == 1], want[taken == 1])
    _check(oracle, queues, b, orders, 128, dims)


@pytest.fixture(scope="module")
def window(tmp_path_factory):
    d = _program(tmp_path_factory, "window")

    def run(most, lengths):
        """-> the scenarios of a window of 512 in the order in which its turns take them, 16 each."""
        (d / "in").write_bytes(np.ascontiguousarray(lengths, dtype=np.uint32).tobytes())
        p = subprocess.run([str(d / "window"), str(most), str(d / "in"), str(d / "out")], capture_output=True, text=True, timeout=60)
        assert p.returncode == 0 and p.stdout == "ran\n", (p.returncode, p.stdout[-500:])
        taken = np.fromfile(d / "out", dtype=np.uint32)
        count = int((lengths != 0).sum())
        assert len(taken) == -(-count // 16) * 16 and (taken[count:] == 0xffffffff).all()
        return taken[:count].astype(int)

    def turns(n):
        """-> window, turn and turns of the window of every workgroup of a batch of n."""
        p = subprocess.run([str(d / "window"), "turns", str(n), str(d / "out")], capture_output=True, text=True, timeout=60)
        assert p.returncode == 0 and p.stdout == "ran\n", (p.returncode, p.stdout[-500:])
        return np.fromfile(d / "out", dtype=np.uint32).reshape(-1, 3).astype(int)

    def marked(b, is_marked, dims):
        """-> {turn: its scenarios} of the turns of a batch of one window that have marks."""
        (d / "in").write_bytes(b.ndims.tobytes() + np.ascontiguousarray(b.npus, np.uint32).tobytes() +
                               np.ascontiguousarray(b.chunks, np.uint32).tobytes() + is_marked.astype(np.uint8).tobytes())
        p = subprocess.run([str(d / "window"), "marked", str(b.n), str(b.max_chunks), str(dims), str(d / "in"), str(d / "out")],
                           capture_output=True, text=True, timeout=60)
        assert p.returncode == 0 and p.stdout == "ran\n", (p.returncode, p.stdout[-500:])
        rows = np.fromfile(d / "out", dtype=np.uint32).reshape(-1, 17)
        return {int(r[0]): [int(v) for v in r[1:] if v != 0xffffffff] for r in rows}

    run.turns, run.marked = turns, marked
    return run


@pytest.mark.parametrize("max_chunks", [1, 8, 24, 64, 90, 250, 512])
@pytest.mark.parametrize("members", [0, 1, 17, 300, 512])
def test_turns_of_a_window_are_the_longest_first(window, max_chunks, members):
    """64 lengths apart where the largest there can be is a power of two (64 chunks: 8 events),
    33 at least; those of a length as they come; the largest length itself among them."""
    rng = np.random.default_rng(members + max_chunks)
    most = 8 * max_chunks
    lengths = np.zeros(512, np.uint32)
    at = np.sort(rng.permutation(512)[:members])
    lengths[at] = rng.integers(1, most + 1, members)
    lengths[at[:1]] = most
    taken = window(most, lengths)
    assert np.array_equal(np.sort(taken), at)
    width = 1
    while 64 * width < most:
        width *= 2
    bucket = np.minimum(lengths[taken].astype(int) // width, 63)
    assert np.array_equal(taken, sorted(at, key=lambda i: (-min(int(lengths[i]) // width, 63), i))), (bucket, width)


@pytest.mark.parametrize("n", [1, 16, 511, 512, 513, 1040, 5003, 60000, 65536, 250001])
def test_every_turn_has_a_workgroup_and_long_ones_are_spread(window, n):
    """Each turn of each window once; of the turns of a window those 1, 2, 4 or 8 apart in the
    order in which they start are of middle length together."""
    turns = window.turns(n)
    of = np.minimum(n - np.arange(-(-n // 512)) * 512, 512)
    assert len(turns) == -(-n // 16)
    assert sorted(map(tuple, turns[:, :2].tolist())) == [(w, t) for w, m in enumerate(of) for t in range(-(-int(m) // 16))]
    assert np.array_equal(turns[:, 2], -(-of[turns[:, 0]] // 16))
    whole = turns[:n // 512 * 32, 1].reshape(32, -1)   # (by place, window)
    for step in (1, 2, 4, 8):
        for first in range(step if whole.size else 0):
            assert (2 * whole[first::step].sum(axis=0) == 31 * 32 // step).all(), (step, first)


@pytest.mark.parametrize("n,others,max_chunks", [(512, 8, 64), (512, 1, 64), (512, 100, 24), (512, 383, 64),
                                                 (512, 512, 128), (300, 40, 250), (17, 3, 512), (17, 16, 512)])
@pytest.mark.parametrize("dims", [3, 4])
@pytest.mark.parametrize("first", ["", "o", "p"])
def test_a_few_marked_scenarios_share_turns(window, first, dims, n, others, max_chunks):
    """Scenarios of other NPU counts, or powers of two, in as few turns as hold them, however
    few they are; else all in one order.  The longest first, and only turns with marks."""
    from paper_2110_04478_amd import workloads
    rng = np.random.default_rng(n + others)
    b = workloads.mixed(n, seed=n + others, max_chunks=max_chunks)
    b.ndims[:] = dims
    at = rng.permutation(n)[:others]
    b.npus[:, at] = 2 * rng.integers(1, 20, (4, others)) + 1
    is_other = np.isin(np.arange(n), at)
    left = ~is_other if first == "p" else is_other
    width, count = 1, int(left.sum())
    while 64 * width < 16 * max_chunks:
        width *= 2
    turns = window.marked(b, left, str(dims) + first)
    taken = [i for t in sorted(turns) for i in turns[t]]
    assert set(np.flatnonzero(left)) <= set(taken)
    if first:
        assert sorted(turns) == list(range(-(-count // 16))) and left[taken[:count]].all()
        taken = taken[:count]
    assert (np.diff(2 * dims * b.chunks.astype(int)[taken]) <= width).all()
    one = np.arange(n) == rng.integers(n)
    assert [int(np.flatnonzero(one)[0]) in v for v in window.marked(b, one, str(dims) + first).values()] == [True]
    assert window.marked(b, np.zeros(n, bool), str(dims) + first) == {} == window.marked(b, left, str(7 - dims) + first)


TABLES = """
#include "themis_quad.hpp"
using namespace themis;
constexpr QuadStages kTables = quad_stages();
constexpr bool copied_words_are_the_tables() {
  for (uint32_t i = 0; i < 512u; ++i)
    if (quad_stage_word(kTables, i) != kTables.v[i]) return false;
  return true;
}
static_assert(copied_words_are_the_tables(), "");
static_assert(sizeof(kTables.v) == 2048u, "");
int main() { return 0; }
"""


def test_the_stage_tables_are_copied_inside_their_array(tmp_path):
    """The copy to LDS takes both tables in one go.  The compiler evaluates it as a
    constant here, for every word: a read beyond the end of an array, also into the one that
    happens to follow it, is an error there."""
    _headers(tmp_path)
    (tmp_path / "tables.cpp").write_text(TABLES)
    p = subprocess.run(["g++", "-std=c++17", "-fsyntax-only", "-w", "-I", str(tmp_path), "-I", os.path.join(HERE, "..", "include"),
                        str(tmp_path / "tables.cpp")], capture_output=True, text=True)
    assert p.returncode == 0, p.stderr[-2000:]


PROBE = """
#include "themis_quad.hpp"
using namespace themis;
__global__ void probe(double* t, const Scenario* s, const FastScenario* fs) {
  using L = LayoutQuad<512, 16>;
  __shared__ uint32_t block[QuadPow2<L, true>::kBytes / 4u];
  QuadQueue<L> queue(block);
  for (uint32_t c = 0; c < s->C; ++c) queue.add(c);
  const Pow2Model m(*s, *fs, true);
  t[threadIdx.x] = simulate_quad<L, false>(QuadPow2<L, true>(*s, m, threadIdx.x & 3u, block), queue, 0u, s->C, 1.0,
                                           [](uint32_t, uint32_t) {}).t_done;
}
"""


def test_links_and_list_ends_may_alias_each_other(tmp_path):
    """A list's ends are written as a word and, where a chunk leaves, as its lower half: the
    compiler must not take the two for accesses to different objects (in the
    intermediate code of such a kernel every access to LDS is one that may alias
    anything)."""
    from paper_2110_04478_amd.csrc import build
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc here")
    (tmp_path / "probe.hip").write_text(PROBE)
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    text = subprocess.run([build.HIPCC, *flags, "-S", "-emit-llvm", "--cuda-device-only", "-o", "-",
                           str(tmp_path / "probe.hip")], check=True, capture_output=True, text=True).stdout
    accesses = re.findall(r"(?:load|store) i(?:16|32) ?.*addrspace\(3\).*", text)
    assert len(accesses) >= 5, len(accesses)
    for a in accesses:
        tag = re.search(r"!tbaa (!\d+)", a)
        access = tag and re.search(r"^%s = !\{(!\d+)," % re.escape(tag.group(1)), text, re.M).group(1)
        kind = access and re.search(r'^%s = !\{!"([^"]*)"' % re.escape(access), text, re.M).group(1)
        assert kind in (None, "omnipotent char"), (kind, a)
