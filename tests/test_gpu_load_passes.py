"""The fused passes of graph load and levelization at their edges, through
the C-ABI against the oracle: sizes around the tiles and chunks they cut a
graph into, task ids in random order (more chain crossings between tiles
than one workgroup ranks), arrays on the host, on the device and on the
device at odd addresses, and the errors of each pass, which come back
together."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2006_03318_amd import binding as B
from paper_2006_03318_amd import workloads as W
from tests import helpers as H
from tests.gpu_common import assert_equal_arrays, gpu_run, require_gpu, say

pytestmark = pytest.mark.gpu


def _graph(rng, n, T, shuffle=False):
    g = W.random_graph_sparse(rng, n, T, mean_in=0.4, window=300, n_edge_cls=2, run_len=20)
    if not shuffle:
        return g
    new = rng.permutation(n)                  # task u becomes new[u]
    dst = np.repeat(np.arange(n), np.diff(g.in_ptr))
    src, dst = new[g.in_src], new[dst]
    o = np.argsort(dst, kind="stable")
    ptr = np.zeros(n + 1, np.int64)
    np.add.at(ptr, dst + 1, 1)
    old = np.empty(n, np.int64)
    old[new] = np.arange(n)
    prev = g.thread_prev[old]
    g.thread_prev = np.where(prev >= 0, new[prev], -1).astype(np.int32)
    for f in ("thread_id", "dur", "gap", "node_cls"):
        setattr(g, f, getattr(g, f)[old])
    g.in_ptr, g.in_src, g.edge_cls = np.cumsum(ptr), src[o].astype(np.int32), g.edge_cls[o]
    return g


@pytest.mark.parametrize("n,T,shuffle", [
    (1, 1, False), (255, 3, False), (1024, 2, False), (1025, 5, False), (2049, 70, False),
    (5000, 4, True), (30_000, 20, True), (262_145, 3, False), (300_000, 300, False)])
def test_sizes_and_id_orders(n, T, shuffle):
    require_gpu()
    rng = np.random.default_rng(700_000 + n + T)
    g = _graph(rng, n, T, shuffle)
    vs = W.random_variants(rng, g, 5, p_remove=0.2)
    say("load passes n=%d T=%d shuffled=%d" % (n, T, shuffle))
    S, F, M = gpu_run(g, vs)
    oS, oF, oM, _ = O.run(g, vs)
    assert_equal_arrays("makespan", M, oM)
    assert_equal_arrays("finish", F, oF)
    assert_equal_arrays("start", S, oS)


def _load(g, where, **bad):
    """dd_graph_load with every array on the host, on the device, or on the
    device one byte off its alignment."""
    import torch
    a = dict(in_ptr=g.in_ptr, in_src=g.in_src, edge_cls=g.edge_cls, thread_prev=g.thread_prev,
             thread_id=g.thread_id, dur=g.dur, gap=g.gap, node_cls=g.node_cls)
    a.update(bad)
    keep, ptr = [], []
    for x in a.values():
        x = np.ascontiguousarray(x)
        if where == "host":
            keep.append(x)
            ptr.append(x.ctypes.data)
        else:
            shift = 1 if where == "odd" else 0
            t = torch.zeros(x.nbytes + 8, dtype=torch.uint8, device="cuda")
            t[shift:shift + x.nbytes] = torch.from_numpy(x.view(np.uint8).reshape(-1)).cuda()
            torch.cuda.synchronize()
            keep.append(t)
            ptr.append(t.data_ptr() + shift)
    import ctypes
    out = ctypes.c_void_p()
    rc = B.lib().dd_graph_load(g.n, g.n_threads, *ptr, None, ctypes.byref(out))
    return rc, out


@pytest.mark.parametrize("where", ["host", "device", "odd"])
def test_where_the_arrays_are(where):
    import torch
    require_gpu()
    rng = np.random.default_rng(710_000)
    g = _graph(rng, 3000, 7)
    want = O.steps(g)[1]
    rc, h = _load(g, where)
    assert rc == B.DD_OK, B.dd_last_error()
    s, _ = B.dd_levelize(h, 3, B.DD_PHASES)
    steps = torch.empty(g.n, dtype=torch.int32, device="cuda")
    B.dd_sched_task_steps(s, steps)
    B.dd_sched_free(s)
    B.dd_graph_free(h)
    assert_equal_arrays("phases", steps.cpu().numpy(), want)


@pytest.mark.parametrize("where", ["host", "device"])
def test_errors_of_every_pass(where):
    require_gpu()
    rng = np.random.default_rng(720_000)
    g = _graph(rng, 3000, 4)
    ordered = [u for u in range(g.n) if g.thread_id[u] == 0]

    def changed(name, at, value):
        a = getattr(g, name).copy()
        a[at] = value
        return {name: a}
    cases = [
        (changed("thread_id", 5, 4), B.DD_EINVAL), (changed("dur", 7, -1), B.DD_EINVAL),
        (changed("gap", 7, 1 << 62), B.DD_ERANGE), (changed("in_src", 3, g.n), B.DD_EINVAL),
        (changed("edge_cls", 3, 64), B.DD_EINVAL), (changed("in_ptr", 1, -2), B.DD_EINVAL),
        (changed("in_ptr", 0, 1), B.DD_EINVAL),
        (changed("thread_prev", ordered[9], ordered[3]), B.DD_ECHAIN),
        (changed("thread_prev", ordered[9], -1), B.DD_ECHAIN),
        (changed("thread_prev", ordered[0], ordered[-1]), B.DD_ECHAIN),
        (changed("thread_prev", ordered[9], g.n), B.DD_EINVAL)]
    dst = int(np.nonzero(np.diff(g.in_ptr) > 0)[0][0])
    k = int(g.in_ptr[dst])
    later = int(np.nonzero(g.thread_id == g.thread_id[dst])[0][-1])
    cases.append((changed("in_src", k, dst), B.DD_ECYCLE))
    if later != dst:
        cases.append((changed("in_src", k, later), B.DD_ECYCLE))
    for bad, want in cases:
        say("load error", where, list(bad))
        rc, h = _load(g, where, **bad)
        assert rc == want and not h.value, (list(bad), rc, want, B.dd_last_error())
    rc, h = _load(g, where)                   # and the next load is not affected
    assert rc == B.DD_OK
    B.dd_graph_free(h)


def test_arrays_written_during_the_load():
    """A caller that writes its device arrays while a load reads them gets a
    graph or an error, never an index outside of the copies: whatever the
    passes check is what they keep.  (The arrays' lengths, in_ptr[n], hold.)"""
    import ctypes

    import torch
    require_gpu()
    rng = np.random.default_rng(730_000)
    g = _graph(rng, 40_000, 6)
    good = dict(in_ptr=g.in_ptr, in_src=g.in_src, edge_cls=g.edge_cls, thread_prev=g.thread_prev,
                thread_id=g.thread_id, dur=g.dur, gap=g.gap, node_cls=g.node_cls)
    bad = {k: v.copy() for k, v in good.items()}
    bad["in_ptr"][1:-1] = rng.integers(-2**40, 2**40, g.n - 1)
    for k in ("in_src", "thread_prev", "thread_id"):
        bad[k][:] = rng.integers(-2**31, 2**31, bad[k].size)
    bad["edge_cls"][:] = 255
    t = {k: torch.from_numpy(np.ascontiguousarray(v)).cuda() for k, v in good.items()}
    tg = {k: v.clone() for k, v in t.items()}
    tb = {k: torch.from_numpy(np.ascontiguousarray(v)).cuda() for k, v in bad.items()}
    torch.cuda.synchronize()
    writer, loader = torch.cuda.Stream(), torch.cuda.Stream()
    codes = set()
    for k in ("in_src", "in_ptr", "thread_id", "thread_prev", "edge_cls"):
        say("load while", k, "is written")
        for _ in range(10):
            with torch.cuda.stream(writer):
                for _ in range(20):
                    t[k].copy_(tb[k])
                    t[k].copy_(tg[k])
            out = ctypes.c_void_p()
            rc = B.lib().dd_graph_load(g.n, g.n_threads, *(x.data_ptr() for x in t.values()),
                                       loader.cuda_stream, ctypes.byref(out))
            codes.add(rc)
            assert rc in (B.DD_OK, B.DD_EINVAL, B.DD_ECYCLE, B.DD_ECHAIN), B.dd_last_error()
            B.dd_graph_free(out)
        torch.cuda.synchronize()
    rc, h = _load(g, "device")
    assert rc == B.DD_OK, B.dd_last_error()
    B.dd_graph_free(h)


def test_backward_dependencies_in_every_workgroup():
    """Each workgroup of the pass that counts the cross-thread edges finds
    errors while others start: the load ends with the error, every time."""
    require_gpu()
    rng = np.random.default_rng(740_000)
    g = _graph(rng, 300_000, 3)
    tail = np.full(3, -1)
    tail[g.thread_id] = np.arange(g.n)                    # the last task of each thread
    deps = np.diff(g.in_ptr) > 0
    deps[tail] = False
    src = g.in_src.copy()
    src[g.in_ptr[:-1][deps]] = tail[g.thread_id[deps]]
    for _ in range(5):
        rc, h = _load(g, "device", in_src=src)
        assert rc == B.DD_ECYCLE and not h.value, B.dd_last_error()


def test_offsets_that_go_back_and_forth():
    """in_ptr that names all edges for every other task: refused by the pass
    that reads it, without going through tasks x edges."""
    require_gpu()
    rng = np.random.default_rng(750_000)
    g = _graph(rng, 200_000, 4)
    ptr = np.zeros(g.n + 1, np.int64)
    ptr[1::2] = g.n_edges
    ptr[-1] = g.n_edges
    for where in ("host", "device"):
        rc, h = _load(g, where, in_ptr=ptr)
        assert rc == B.DD_EINVAL and not h.value, B.dd_last_error()


@pytest.mark.parametrize("fan", [7, 8, 9, 15, 16, 17, 1000])
def test_many_dependencies_of_one_task(fan):
    """Lists around the eight edges that are loaded together, from its own
    thread and from others, of both classes; a bad entry anywhere is found."""
    require_gpu()
    rng = np.random.default_rng(760_000 + fan)
    m = max(40, fan)
    thread = rng.integers(0, 4, m).tolist() + [0, 1, 2]
    edges = [(int(s), d) for d in (m, m + 1, m + 2) for s in rng.permutation(m)[:fan]]
    g = H.graph(4, thread, edges, rng.integers(0, 900, m + 3), rng.integers(0, 90, m + 3),
                edge_cls=rng.integers(0, 2, len(edges)), n_edge_cls=2)
    vs = W.random_variants(rng, g, 5, p_remove=0.2)
    S, F, M = gpu_run(g, vs)
    oS, oF, oM, _ = O.run(g, vs)
    assert_equal_arrays("makespan", M, oM)
    assert_equal_arrays("finish", F, oF)
    for where in ("host", "device"):
        for k in range(fan, 2 * fan, max(1, fan // 20)):
            src, cls = g.in_src.copy(), g.edge_cls.copy()
            src[k], cls[k] = -1, 64
            assert _load(g, where, in_src=src)[0] == B.DD_EINVAL
            assert _load(g, where, edge_cls=cls)[0] == B.DD_EINVAL
