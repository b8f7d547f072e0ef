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


def _late(seed, n, fan, at, parents=1, V=5, max_dur=1000):
    """A graph as in _case with `fan` more tasks on its last thread, each of
    which waits for task `at` and (parents > 1) for tasks after it."""
    g, vs, pp, prio = _case(seed, n, V=V, max_dur=max_dur)
    ps = np.minimum(at + 3 * np.arange(parents), n - 1)
    rep = lambda a, v: np.r_[a, np.full(fan, v)].astype(a.dtype)
    g2 = W.TaskGraph(n + fan, g.n_threads, np.r_[g.in_ptr, g.in_ptr[-1] + parents * (1 + np.arange(fan))],
                     np.r_[g.in_src, np.tile(ps, fan)].astype(np.int32), np.r_[g.edge_cls, np.zeros(fan * parents, np.uint8)],
                     rep(g.thread_prev, -1), rep(g.thread_id, g.n_threads - 1), rep(g.dur, 7), rep(g.gap, 1),
                     rep(g.node_cls, 0), g.n_node_cls, g.n_edge_cls, rep(g.kind, 0), rep(g.layer, -1),
                     rep(g.launch_of, -1), "late")
    rng = np.random.default_rng(seed + 1)
    return g2, W.random_variants(rng, g2, V, p_remove=0.2), rep(pp, 1), np.r_[prio, rng.integers(-2, 3, fan)].astype(np.int32)


@pytest.mark.parametrize("policy", [0, 1])
@pytest.mark.parametrize("at,parents,V", [(0, 1, 3), (1, 2, 9), (63, 1, 5), (64, 3, 5), (300, 1, 33), (700, 2, 257),
                                          (890, 1, 2049), (899, 1, 5)])
def test_goes_on_where_it_stopped(policy, at, parents, V):
    """300 tasks become ready, or begin to wait, late in the run: the general
    kernel goes on from there, in every variant from its own place."""
    require_gpu()
    g, vs, pp, prio = _late(7000 + at, 900, 300, at, parents, V)
    _check(g, vs, policy, pp, prio, "late%d" % at)


@pytest.mark.parametrize("policy", [0, 1])
def test_some_variants_stop_and_others_end(policy):
    """A task that lasts longer than 32-bit differences hold in the variants
    that stretch it; the others run past it, or have ended, when they hear."""
    require_gpu()
    for u, n in ((40, 400), (390, 400), (20, 3000), (2990, 3000)):
        g, _, pp, prio = _case(n + u, n, n_cls=2, max_dur=10**6)
        g.node_cls[:] = 0
        g.node_cls[u] = 1
        g.dur[u] = 1 << 31
        vs = H.variants(g, scales=[{}, {1: (2, 1)}, {1: (1, 8)}, {1: (3, 1), 0: (1, 2)}, {1: (0, 1)}] * 4)
        _check(g, vs, policy, pp, prio, "some%d" % u)


def test_errors_after_going_on():
    """Past the registers, a cycle and a frontier beyond the capacity."""
    from paper_2006_03318_amd import batch as BT
    from paper_2006_03318_amd import binding as B
    require_gpu()
    g, vs, pp, prio = _late(7100, 900, 300, 500)
    g.in_src[-1], g.in_src[-2] = g.n - 2, g.n - 1         # the last two tasks wait for each other
    with pytest.raises(B.DDError) as ei:
        BT.simulate_policy(g, vs, 1, pp, prio)
    assert ei.value.code == B.DD_ECYCLE
    g, vs, pp, prio = _late(7200, 900, 1100, 500)
    with pytest.raises(B.DDError) as ei:
        BT.simulate_policy(g, vs, 1, pp, prio)
    assert ei.value.code == B.DD_ELIMIT


def test_a_call_does_not_pay_for_both_kernels():
    """A graph that outgrows the registers at its end takes no longer than the
    general kernel takes for all of it (which runs where threads number 65)."""
    import time

    import torch
    from paper_2006_03318_amd import binding as B
    require_gpu()
    g, vs, pp, prio = _late(7300, 4000, 400, 3990, V=30)

    def seconds(n_threads):
        t = lambda a, d: torch.from_numpy(np.ascontiguousarray(a).astype(d)).cuda()
        h = B.dd_graph_load_ex(g.n, n_threads, t(g.in_ptr, np.int64), t(g.in_src, np.int32), None, t(g.thread_prev, np.int32),
                               t(g.thread_id, np.int32), t(g.dur, np.int64), t(g.gap, np.int64), t(g.node_cls, np.uint16),
                               B.DD_LOAD_SHARED_THREADS)
        var = B.dd_apply_transforms(h, 30, int(vs.scale.shape[0]), t(vs.scale, np.int32), t(vs.remove_bits, np.uint32), None)
        fin = torch.empty((g.n, 30), dtype=torch.int64, device="cuda")
        ms = torch.empty(30, dtype=torch.int64, device="cuda")
        ppd, prd = t(pp, np.uint8), t(prio, np.int32)
        best = []
        for _ in range(6):
            torch.cuda.synchronize()
            at = time.perf_counter()
            B.dd_simulate_policy(h, var, B.DD_POLICY_PRIORITY, ppd, prd, fin, None, ms)
            best.append(time.perf_counter() - at)
        B.dd_variants_free(var)
        B.dd_graph_free(h)
        return min(best), fin.cpu().numpy()
    (late, f0), (general, f1) = seconds(g.n_threads), seconds(65)
    assert np.array_equal(f0, f1)
    assert late < 1.25 * general, (late, general)
