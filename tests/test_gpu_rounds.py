"""Levelization rounds with 17 and more threads: the schedule, seen through
the simulation's exact results, where segments and steps outgrow the LDS they
wait in, where a task has dozens of parents that finish one after another, and
where a ready run is longer than the probes and than one step of the scan."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2006_03318_amd import workloads as W
from tests import helpers as H
from tests.gpu_common import assert_equal_arrays, gpu_run, require_gpu, say

pytestmark = pytest.mark.gpu


def _check(g, label):
    say("rounds", label, "n=%d T=%d" % (g.n, g.n_threads))
    vs = W.random_variants(np.random.default_rng(g.n), g, 3, p_remove=0.1)
    S, F, M = gpu_run(g, vs)
    oS, oF, oM, _ = O.run(g, vs)
    assert_equal_arrays("makespan", M, oM)
    assert_equal_arrays("finish", F, oF)
    assert_equal_arrays("start", S, oS)


@pytest.mark.parametrize("T", [17, 32, 33, 64, 65, 256])
@pytest.mark.parametrize("mean_in,window,run_len", [(0.5, 40, 1), (6.0, 3000, 1), (0.02, 9000, 30)])
def test_random(T, mean_in, window, run_len):
    """Thousands of short steps, many parents on many threads, long runs."""
    require_gpu()
    rng = np.random.default_rng(T + int(100 * mean_in))
    _check(W.random_graph_sparse(rng, 12_000, T, mean_in=mean_in, window=window, run_len=run_len, n_edge_cls=2),
           "random")


@pytest.mark.parametrize("T", [20, 64, 65])
@pytest.mark.parametrize("run", [127, 128, 129, 1024, 4096, 4097, 9000])
def test_long_run_and_joins(T, run):
    """Thread 1 waits task by task for thread 0 (one run of `run` candidates),
    then a chain through the other threads, and a task that waits for each of
    them and lies between others on its thread."""
    require_gpu()
    thread, edges = [], []
    for i in range(run):
        thread.append(0)
    for i in range(run):
        thread.append(1)
        edges.append((i, run + i))
    links = []
    for t in range(2, T):
        links.append(len(thread))
        thread.append(t)
        edges.append((links[-2] if len(links) > 1 else 2 * run - 1, links[-1]))
    for k in range(3):                        # joins, each after the last on thread 0
        j = len(thread)
        thread.append(0)
        edges += [(u, j) for u in links]
        edges.append((2 * run - 1, j))
    rng = np.random.default_rng(run + T)
    n = len(thread)
    edges.sort(key=lambda e: (e[1], e[0]))
    _check(H.graph(T, thread, edges, rng.integers(0, 90, n).tolist(), rng.integers(0, 9, n).tolist()), "joins")
