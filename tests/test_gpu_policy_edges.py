"""The schedule-rule kernel that keeps its state in registers, at the edges of
what it takes: bit-exact against the oracle where its window of task records
moves and children lie outside of it, where times pass its 32-bit base, at its
limits of threads, classes, ready and waiting tasks, and just past each of
them, where the general kernel takes over."""
import numpy as np
import pytest

from paper_2006_03318_amd import workloads as W
from tests import helpers as H
from tests.gpu_common import require_gpu
from tests.test_gpu_policy import _check

pytestmark = pytest.mark.gpu


def _case(seed, n, threads=4, V=9, n_cls=3, max_dur=1000):
    """Ordered and shared threads (whose tasks nearly all follow an earlier one,
    so that few are ready at once); every edge class on, as the kernel asks."""
    rng = np.random.default_rng(seed)
    g, pp, prio = W.random_shared_graph(rng, n, threads - threads // 2, threads // 2, mean_in=1.3,
                                        window=48, chain_frac=0.95, n_node_cls=n_cls, max_dur=max_dur)
    return g, W.random_variants(rng, g, V, p_remove=0.2), pp, prio


def _side_by_side(seed, n, V):
    """Two graphs of n / 2 tasks that run at the same time, on threads of their
    own: a task in the second is n / 2 ids past what runs with it."""
    rng = np.random.default_rng(seed)
    h = n // 2
    parts = [W.random_shared_graph(rng, h, 2, 2, mean_in=1.3, window=48, chain_frac=0.95) for _ in range(2)]
    (a, app, apr), (b, bpp, bpr) = parts
    prev = np.r_[a.thread_prev, np.where(b.thread_prev < 0, -1, b.thread_prev + h)].astype(np.int32)
    g = W.TaskGraph(2 * h, 8, np.r_[a.in_ptr, b.in_ptr[1:] + a.in_ptr[-1]], np.r_[a.in_src, b.in_src + h].astype(np.int32),
                    np.r_[a.edge_cls, b.edge_cls], prev, np.r_[a.thread_id, b.thread_id + 4].astype(np.int32),
                    np.r_[a.dur, b.dur], np.r_[a.gap, b.gap], np.r_[a.node_cls, b.node_cls], a.n_node_cls,
                    a.n_edge_cls, np.r_[a.kind, b.kind], np.r_[a.layer, b.layer], np.r_[a.launch_of, b.launch_of],
                    "side-by-side")
    return g, W.random_variants(rng, g, V, p_remove=0.2), np.r_[app, bpp], np.r_[apr, bpr]


@pytest.mark.parametrize("policy", [0, 1])
@pytest.mark.parametrize("make,n,V", [(_case, 4096, 5), (_case, 4097, 5), (_case, 6000, 3), (_case, 700, 257),
                                      (_case, 700, 2049), (_case, 1, 33), (_side_by_side, 4400, 17),
                                      (_side_by_side, 6000, 17)])
def test_window(policy, make, n, V):
    """Whole graphs in the window, one task more, and tasks outside of it; one
    variant and eight to a workgroup, with a remainder."""
    require_gpu()
    g, vs, pp, prio = make(n + V, n, V=V)
    _check(g, vs, policy, pp, prio, "window")


@pytest.mark.parametrize("policy", [0, 1])
@pytest.mark.parametrize("threads,n_cls", [(2, 1), (64, 3), (65, 3), (5, 512), (5, 513)])
def test_threads_and_classes(policy, threads, n_cls):
    require_gpu()
    g, vs, pp, prio = _case(threads + n_cls, 700, threads=threads, n_cls=n_cls)
    _check(g, vs, policy, pp, prio, "threads%d-classes%d" % (threads, n_cls))


@pytest.mark.parametrize("policy", [0, 1])
@pytest.mark.parametrize("ready", [255, 256, 257])
def test_ready_tasks(policy, ready):
    """As many tasks ready at once as the registers hold, and one more."""
    require_gpu()
    n = ready
    g = H.graph(1, [0] * n, [], list(range(1, n + 1)), [0] * n, thread_order=[])
    g.thread_prev = np.full(n, -1, np.int32)
    pp = (np.arange(n) % 3 != 0).astype(np.uint8)
    prio = (np.arange(n) % 5 - 2).astype(np.int32)
    _check(g, H.variants(g, V=3), policy, pp, prio, "ready%d" % ready)


@pytest.mark.parametrize("policy", [0, 1])
@pytest.mark.parametrize("waiting,parents", [(255, 2), (256, 2), (257, 2), (40, 6), (40, 7), (40, 9)])
def test_waiting_tasks(policy, waiting, parents):
    """As many tasks with a part of their parents done as the registers hold,
    and one more; parents around the number that an out-edge can carry."""
    require_gpu()
    # thread 0: `parents` tasks in a row, each a parent of every waiting task
    n = parents + waiting
    edges = [(p, parents + w) for w in range(waiting) for p in range(parents)]
    rng = np.random.default_rng(waiting + parents)
    g = H.graph(2, [0] * parents + [1] * waiting, edges, rng.integers(1, 50, n).tolist(), [0] * n,
                thread_order=[list(range(parents))])
    g.thread_prev = np.array([-1] + list(range(parents - 1)) + [-1] * waiting, np.int32)
    pp = np.r_[np.zeros(parents, np.uint8), np.ones(waiting, np.uint8)]
    _check(g, H.variants(g, V=3), policy, pp, rng.integers(-2, 3, n).astype(np.int32), "waiting")


@pytest.mark.parametrize("policy", [0, 1])
@pytest.mark.parametrize("max_dur", [10**6, 10**8, 1 << 30, (1 << 32) - 1, 1 << 33])
def test_long_times(policy, max_dur):
    """Times far past 32 bits: the base moves, and where one task lasts longer
    than the differences hold, or 2^32 and more, the general kernel runs."""
    require_gpu()
    g, vs, pp, prio = _case(max_dur % 1009, 900, max_dur=max_dur)
    _check(g, vs, policy, pp, prio, "long")
    vs = H.variants(g, V=2)
    _check(g, vs, policy, pp, prio, "long-unscaled")
