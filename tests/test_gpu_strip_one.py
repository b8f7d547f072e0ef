"""The strip kernel with one variant per workgroup against the oracle (start,
finish and makespan bit-exact).  dd_simulate_batch and dd_simulate_batch_vs
take the one-variant kernel for nearly all such calls; this instance serves
dd_simulate_batch_noalloc with up to 256 variants, calls whose times, scales
or classes that kernel does not hold, and calls without room for its scratch.
Its double and its int64 form, both sides of the bounds between them, thread
carries and gathered predecessors, long lists of parents, both step modes."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2006_03318_amd import batch as BT
from paper_2006_03318_amd import binding as B
from paper_2006_03318_amd import workloads as W
from tests import test_gpu_time_arith as TA
from tests.gpu_common import assert_equal_arrays, require_gpu, say
from tests.test_gpu_coverage import _fan_in_graph, _multi_fan_in

pytestmark = pytest.mark.gpu


def _check(g, vs, label, mode=B.DD_PHASES, fp=None):
    import torch
    assert vs.n_variants <= 256              # one variant per workgroup
    if fp is not None:
        bound, dp = TA._bounds(g, vs)
        assert (bound < TA.FP_LIMIT and dp < 2**53) == fp, (bound, dp)
    di = BT.to_device(g, vs)
    gh = BT.load_graph(di)
    oS, oF, oM, _ = O.run(g, vs)
    for v0, v1, mask, scale, rm, on in di.batches:
        sch, _ = B.dd_levelize(gh, mask, mode)
        var = B.dd_apply_transforms(gh, v1 - v0, di.n_cls, scale, rm, on)
        for start in (True, False):
            say("strip of one", label, "n=%d threads=%d V=%d start=%d" % (g.n, g.n_threads, v1 - v0, start))
            fin = torch.full((g.n, v1 - v0), -1, dtype=torch.int64, device="cuda")
            st = torch.full_like(fin, -1) if start else None
            ms = torch.full((v1 - v0,), -1, dtype=torch.int64, device="cuda")
            B.dd_simulate_batch_noalloc(gh, sch, var, fin, st, ms)
            assert_equal_arrays(label + " makespan", ms.cpu().numpy(), oM[v0:v1])
            assert_equal_arrays(label + " finish", fin.cpu().numpy().T, oF[v0:v1])
            if start:
                assert_equal_arrays(label + " start", st.cpu().numpy().T, oS[v0:v1])
        B.dd_sched_free(sch)
        B.dd_variants_free(var)
    B.dd_graph_free(gh)


@pytest.mark.parametrize("V", [1, 37, 256])
@pytest.mark.parametrize("threads", [3, 64, 65, 700])
def test_uniform(V, threads):
    require_gpu()
    rng = np.random.default_rng(970_000 + V + threads)
    g = W.random_graph_sparse(rng, 4000, threads, mean_in=0.4, window=600, n_edge_cls=2, n_node_cls=20, run_len=12)
    _check(g, TA._uniform_variants(rng, g, V, TA.RATIOS), "uniform", fp=True)


@pytest.mark.parametrize("mode", [B.DD_PHASES, B.DD_LEVELS])
def test_edge_classes_and_quotients(mode):
    require_gpu()
    rng = np.random.default_rng(971_000)
    g = W.random_graph_sparse(rng, 5000, 5, mean_in=0.8, window=150, n_edge_cls=3, n_node_cls=9, run_len=6)
    _check(g, W.random_variants(rng, g, 70, p_remove=0.2), "classes", mode=mode)


@pytest.mark.parametrize("ratios,fp", [([(1, 1), (128, 1), (255, 2), (3, 256), (1, 2)], True),
                                       ([(1, 1), (1024, 1), (2047, 2), (3, 256), (1, 2)], False)])
def test_times_around_the_bound(ratios, fp):
    require_gpu()
    rng = np.random.default_rng(92_000)
    g = TA._long_graph(rng)
    _check(g, TA._uniform_variants(rng, g, 33, ratios, p_remove=0.1, p_scale=0.9), "long", fp=fp)


@pytest.mark.parametrize("p,fp", [((1 << 20) + 1, True), ((1 << 21) + 1, False)])
def test_products_around_the_bound(p, fp):
    require_gpu()
    rng = np.random.default_rng(93_000)
    g = TA._long_graph(rng, n=400, T=3, lo=2**32 - 2**20, hi=2**32 - 1)
    g.dur[7] = 2**32 - 1
    q = 1 << ((p - 1).bit_length() - 1)
    _check(g, TA._uniform_variants(rng, g, 20, [(1, 1), (p, q), (q + 1, q * 2)], p_remove=0.1), "products", fp=fp)


def test_long_lists_of_parents():
    require_gpu()
    rng = np.random.default_rng(94_000)
    g = _fan_in_graph(rng)[0]
    g.node_cls = rng.integers(0, 5, size=g.n).astype(np.uint16)
    g.n_node_cls = 5
    _check(g, TA._uniform_variants(rng, g, 26, TA.RATIOS, p_remove=0.25), "fan-in", fp=True)
    g = _multi_fan_in(rng)
    g = g[0] if isinstance(g, tuple) else g
    _check(g, W.random_variants(rng, g, 37, p_remove=0.2), "fan-ins")
