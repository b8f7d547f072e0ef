"""Parity of the one-variant-per-workgroup kernel with the oracle (start,
finish and makespan bit-exact) where its batches, window and ring can go
wrong: step widths around the limits of a narrow step, of a group of narrow
steps and of a batch; parents older than the ring; five and more parents in
narrow and in wide steps; scale quotients at the limit of the exact
correction; every variant count around a multiple of 8 workgroups.
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2006_03318_amd import batch as BT
from paper_2006_03318_amd import binding as B
from paper_2006_03318_amd import workloads as W
from paper_2006_03318_amd.workloads import VariantSet, pack_bits
from tests import helpers as H
from tests.gpu_common import assert_equal_arrays, gpu_run, require_gpu, say

pytestmark = pytest.mark.gpu


def _check(g, vs, label, mode=B.DD_PHASES, want_start=True):
    say("solo", label, "n=%d threads=%d V=%d" % (g.n, g.n_threads, vs.n_variants))
    S, F, M = gpu_run(g, vs, mode=mode, variants_per_wg=1, want_start=want_start)
    oS, oF, oM, _ = O.run(g, vs, want_start=want_start)
    assert_equal_arrays(label + " makespan", M, oM)
    assert_equal_arrays(label + " finish", F, oF)
    if want_start:
        assert_equal_arrays(label + " start", S, oS)


def _runs(widths, rng, threads=3, extra=0):
    """One run of tasks per step, on threads in turn: the first task of each
    run waits for the last of the run before; `extra` random tasks of each
    run also wait for random tasks of any earlier run."""
    thread, edges, first = [], [], 0
    for r, w in enumerate(widths):
        thread += [r % threads] * w
        if r:
            edges.append((first - 1, first))
            for _ in range(extra):
                edges.append((int(rng.integers(0, first)), first + int(rng.integers(0, w))))
        first += w
    n = len(thread)
    edges = [(a, b) for a, b in edges if thread[a] != thread[b]]
    return H.graph(threads, thread, edges, rng.integers(0, 5000, n), rng.integers(0, 300, n),
                   cls=rng.integers(0, 4, n), edge_cls=rng.integers(0, 2, len(edges)), n_cls=4,
                   n_edge_cls=2)


@pytest.mark.parametrize("widths", [
    [127, 128, 129, 1, 128, 128, 128, 128, 127, 1, 130],   # narrow or not
    [1] * 383 + [128, 1, 1],                                # a full group, then the longest member
    [1] * 384 + [128, 2], [64] * 20, [65, 64, 63] * 9, [383, 1, 385, 2, 384],
    [511, 1, 512, 1, 513, 1, 1023, 1, 1024, 1, 1025], [1], [512], [513], [2, 3000, 5],
])
def test_step_widths(widths):
    require_gpu()
    rng = np.random.default_rng(800 + len(widths))
    g = _runs(widths, rng, extra=3)
    _check(g, W.random_variants(rng, g, 9, p_remove=0.2), "widths")


@pytest.mark.parametrize("V", [1, 7, 8, 9, 33, 63, 65])
def test_variant_counts(V):
    require_gpu()
    rng = np.random.default_rng(820 + V)
    g = _runs([5, 1, 40, 200, 7, 600, 3, 3, 3], rng, extra=4)
    _check(g, W.random_variants(rng, g, V, p_remove=0.3), "V", want_start=V % 2 == 1)


def test_parents_older_than_the_ring():
    """Tasks 33,000 and more positions after their parents (the ring holds
    32,768 releases), in wide and in narrow steps, as first, second and
    further parents, next to parents just inside the ring."""
    require_gpu()
    rng = np.random.default_rng(840)
    n0 = 34000
    thread = [0] * n0 + [1] * 3000 + [2] * 40 + [3] * 700
    edges = [(n0 - 1, n0), (n0 + 2999, n0 + 3000), (n0 + 3039, n0 + 3040)]
    for b in range(n0, len(thread), 7):
        for _ in range(1 + b % 4):
            edges.append((int(rng.integers(0, n0)), b))
    n = len(thread)
    g = H.graph(4, thread, edges, rng.integers(0, 5000, n), rng.integers(0, 300, n),
                cls=rng.integers(0, 3, n), n_cls=3)
    _check(g, W.random_variants(rng, g, 10, p_remove=0.2), "far")


@pytest.mark.parametrize("run", [6, 700])
def test_many_parents(run):
    """A task with 80 parents on 80 threads, some in its own batch, some in
    the one before, some older; in a narrow step and in a wide one."""
    require_gpu()
    rng = np.random.default_rng(860 + run)
    thread, edges = [], []
    for r in range(12):
        base = len(thread)
        for i in range(80):
            thread += [1 + i] * (1 + (r + i) % 3)
        last = {}
        for u in range(base, len(thread)):
            last[thread[u]] = u
        head = len(thread)
        thread += [0] * run
        edges += [(u, head) for u in last.values()]
        edges += [(u, head + run // 2) for u in list(last.values())[:3 + r % 4]]
        if r:
            edges += [(int(rng.integers(0, base)), head + run - 1) for _ in range(5)]
            edges.append((base - 1, base))
    edges = [(a, b) for a, b in edges if thread[a] != thread[b]]
    n = len(thread)
    g = H.graph(81, thread, edges, rng.integers(0, 5000, n), rng.integers(0, 300, n),
                edge_cls=rng.integers(0, 3, len(edges)), n_edge_cls=3)
    _check(g, W.random_variants(rng, g, 17, p_remove=0.2), "many-parents")


def test_scale_quotients():
    """floor(d * p / q) where the rounded product comes closest to an integer:
    products up to 2^50, quotients at and next to multiples of q; and the
    same with products past 2^50, which the strip kernel takes."""
    require_gpu()
    rng = np.random.default_rng(880)
    qs = [3, 7, 10, 641, 65537, 1000003, 2**30 + 3, 2**31 - 1]
    V = 2 * len(qs) + 1
    n = 600
    dur = rng.integers(2**31, 2**32 - 1, n)
    for i, q in enumerate(qs):                        # multiples of q, and one less
        k = (2**32 - 2) // q
        dur[2 * i], dur[2 * i + 1] = k * q, k * q - 1
    g = H.graph(3, rng.integers(0, 3, n), [(i, i + 1) for i in range(n - 1)], dur, np.zeros(n, int))
    for pmax in (2**18 - 1, 2**21 - 1):
        s = np.ones((1, V, 2), np.int32)
        for i, q in enumerate(qs):
            s[0, 2 * i + 1] = (1, q)
            s[0, 2 * i + 2] = (min(q - 1, pmax), q)
        assert int(g.dur.max()) * int(s[..., 0].max()) < 2**32 * (pmax + 1)
        vs = VariantSet(V, s, pack_bits(np.zeros((n, V), bool)), np.full((V, 1), 1, np.uint64),
                        [(0, V, 1)])
        _check(g, vs, "quotients")


def test_plan_and_fallback():
    """Which launch dd_simulate_batch takes around its limits, and the strip
    kernel for times that doubles do not hold."""
    import torch
    require_gpu()
    rng = np.random.default_rng(900)
    wide = _runs([600, 700, 650, 640], rng)           # 647 positions a step
    slim = _runs([8] * 300, rng)
    for g, V, want in ((wide, 768, 1), (wide, 769, 4), (slim, 769, 1), (slim, 2048, 1),
                       (slim, 2049, 16)):
        vs = W.random_variants(rng, g, V, p_remove=0.1)
        res, gh, hs = BT.simulate(BT.to_device(g, vs), keep_handles=True)
        torch.cuda.synchronize()
        assert [B.dd_simulate_plan(s_, v_) for s_, v_ in hs] == [want], (g.n, V)
        ms = torch.cat([r[4] for r in res]).cpu().numpy()
        for s_, v_ in hs:
            B.dd_sched_free(s_)
            B.dd_variants_free(v_)
        B.dd_graph_free(gh)
        assert_equal_arrays("makespan", ms, O.run(g, vs, want_start=False, want_finish=False)[2])
    big = _runs([5, 300, 7], rng)
    big.dur[3] = 2**32                                # past the records' 32 bits
    _check(big, W.random_variants(rng, big, 5, p_remove=0.1), "64-bit durations")
