"""What a user has this framework do, as cases that can be timed.

Each case is one pass through the public entry points, on a trace-shaped
graph of `workloads` (durations drawn from the seed) and a table of what-if
variants of the kinds that `recipes` compiles: mixed precision (1/3 and 1/2),
layer scaling, cheaper launch calls, fused element-wise kernels (removed
with their launches), faster links, gradient compression, memory offloading
policies.  Four paths:

  step       a trace arrives: load the graph, levelize it (once per batch of
             edge classes), build the transform tables, simulate;
  sweep      more questions about a loaded trace: the graph and its schedule
             are kept, the tables are built and simulated;
  breakdown  where each variant's time goes, from a finished simulation;
  policy     the parameter-server graph under a schedule rule, task by task.

All outputs are whole numbers (int64 nanoseconds) and the same for every
correct implementation.
"""
import math
import sys

import numpy as np
import torch

from paper_2006_03318_amd import batch, binding as B, workloads as W

DEV = "cuda"
# per iteration: tasks, dependencies between threads, GPU kernels plus waiting
# calls, waiting calls
SHAPE = {"cnn": (403, 204, 201, 1), "vdnn": (483, 338, 201, 1),
         "transformer": (32768, 16435, 16383, 2), "allreduce": (32815, 16713, 16383, 2),
         "seq2seq": (28835, 14420, 14417, 1), "p3": (459, 420, 78, 1)}
MOST_PAIRS = 1 << 31            # task-variant pairs of the largest case


def listed():
    return [
        # the smallest whole use: a CNN trace of four iterations and a handful of recipes
        dict(name="step_cnn", path="step", model="cnn", iters=4, variants=8, amp=True, start=False),
        # one question about a trace that is already loaded
        dict(name="ask_cnn", path="sweep", model="cnn", iters=4, variants=1, amp=True, start=True),
        # offloading policies as edge classes that differ from variant to variant
        dict(name="sweep_vdnn", path="sweep", model="vdnn", iters=4, variants=256, amp=True, start=False),
        # an ordinary sweep of one transformer iteration
        dict(name="step_transformer", path="step", model="transformer", iters=1, variants=256, amp=True, start=False),
        # data-parallel training: four channel orders, so four schedules, on 51 threads
        dict(name="step_allreduce", path="step", model="allreduce", iters=1, variants=1024, amp=True, start=False),
        # a long trace of small kernels and few variants, start times wanted too
        dict(name="step_seq2seq", path="step", model="seq2seq", iters=9, variants=64, amp=True, start=True),
        # an odd number of variants over a kept schedule of five iterations
        dict(name="sweep_transformer_x5", path="sweep", model="transformer", iters=5, variants=333, amp=True, start=False),
        # the large sweep that bench.py times
        dict(name="step_transformer_x32", path="step", model="transformer", iters=32, variants=2048, amp=False, start=False),
        # the breakdown of an ordinary sweep, and of a large one
        dict(name="breakdown_transformer", path="breakdown", model="transformer", iters=1, variants=256, amp=True, start=False),
        dict(name="breakdown_transformer_x8", path="breakdown", model="transformer", iters=8, variants=1000, amp=True, start=False),
        # schedule rules: a short trace under the default rule, a long one under P3's
        dict(name="policy_earliest", path="policy", model="p3", iters=2, variants=30, amp=True, start=True),
        dict(name="policy_p3", path="policy", model="p3", iters=32, variants=2048, amp=True, start=False),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    path = rng.choices(("step", "sweep", "breakdown", "policy"), (4, 3, 2, 2))[0]
    model = "p3" if path == "policy" else rng.choice(("cnn", "vdnn", "transformer", "allreduce", "seq2seq"))
    iters = _log_int(rng, 1, {"cnn": 64, "vdnn": 64, "transformer": 32, "allreduce": 2, "seq2seq": 12, "p3": 32}[model])
    pairs = MOST_PAIRS if path == "step" else MOST_PAIRS // 4
    variants = _log_int(rng, 4 if model == "allreduce" else 1, min(2048, pairs // (SHAPE[model][0] * iters)))
    return dict(path=path, model=model, iters=iters, variants=variants, amp=rng.random() < 0.7, start=rng.random() < 0.25)


# ---------------------------------------------------------------------------
# inputs
def _graph(case, seed):
    """The trace: (graph, push/pull flags, priorities) with the task classes
    that the variant tables scale."""
    model, iters = case["model"], case["iters"]
    pp = prio = None
    if model == "vdnn":
        g, _ = W.vdnn_workload(iters=iters, variants=1, seed=seed)
    elif model == "p3":
        g, _, pp, prio = W.p3_workload(iters=iters, variants=1, seed=seed)
    else:
        k = {"cnn": 1, "transformer": 5, "allreduce": 3, "seq2seq": 4}[model]
        g, _ = W.config(k, seed=seed, variants=4 if model == "allreduce" else 1, iters=iters)
    bucket = np.zeros(g.n, np.int64)        # the all-reduce of one bucket, in each iteration
    if model == "allreduce":
        for it in range(iters):
            ids = np.nonzero((g.kind == W.K_COMM) & (g.iteration == it))[0]
            bucket[ids] = np.arange(ids.shape[0])
    key = ((g.layer.astype(np.int64) + 1) * 16 + g.kind) * 512 + g.op.astype(np.int64) * 64 + bucket
    _, first, inv = np.unique(key, return_index=True, return_inverse=True)
    g.node_cls = inv.reshape(-1).astype(np.uint16)
    g.n_node_cls = int(first.shape[0])
    return g, first, pp, prio


def _scales(case, g, rep, rng):
    """int32 [classes][V][2]: the (p, q) of every class in every variant
    (variant 0 is the baseline)."""
    V, C = case["variants"], g.n_node_cls
    kind, layer, op = g.kind[rep], g.layer[rep], g.op[rep]
    P, Q = np.ones((C, V), np.int64), np.ones((C, V), np.int64)

    def scale(rows, some, num, den):         # num, den: per variant, or per row and variant
        P[rows] *= np.where(some, num, 1)
        Q[rows] *= np.where(some, den, 1)

    gpu = np.isin(kind, W.GPU_KINDS)
    gemm = gpu & np.isin(kind, (W.K_GEMM, W.K_CONV))
    amp = (rng.random(V) < 0.5) & bool(case["amp"])
    scale(gemm, amp, 1, 3)
    scale(gpu & ~gemm, amp, 1, 2)
    q = 2 ** rng.integers(0, 4, V)
    p = rng.integers(0, 2 * q + 1)
    scaled = rng.random(V) < 0.5
    for l in np.unique(layer[gpu]):
        scale(gpu & (layer == l), scaled & (rng.random(V) < 0.5), p, q)
    ln, ld = np.array([(1, 1), (0, 1), (1, 4), (1, 2), (2, 1)]).T
    pick = rng.integers(0, 5, V)
    scale(kind == W.K_LAUNCH, True, ln[pick], ld[pick])
    comm = kind == W.K_COMM
    if comm.any():
        gbps = rng.choice((10, 25, 100) if case["model"] == "allreduce" else (1, 2, 5, 10, 25, 40), V)
        scale(comm, True, 10, gbps)
        if case["model"] == "allreduce":
            scale(comm, rng.random((int(comm.sum()), V)) < 0.5, 1, 4)
    copies = (kind == W.K_MEMCPY) & np.isin(op, (W.OP_OFFLOAD, W.OP_PREFETCH))
    if copies.any():
        cn, cd = np.array([(1, 1), (1, 2), (2, 1)]).T
        pick = rng.integers(0, 3, V)
        scale(copies, True, cn[pick], cd[pick])
    P[:, 0], Q[:, 0] = 1, 1
    d = np.gcd(P, Q)
    d[d == 0] = 1
    return np.ascontiguousarray(np.stack([P // d, Q // d], axis=2).astype(np.int32))


def _removals(case, g, rng, seed):
    """uint32 [n][ceil(V / 32)] on the GPU: each variant but the baseline drops
    10 to 50 % of the small kernels with their launch calls (seven in ten
    variants), and offloading copies where the policy has none."""
    V = case["variants"]
    Wd = (V + 31) // 32
    dens = np.where(rng.random(V) < 0.7, rng.uniform(0.1, 0.5, V), 0.0)
    dens[0] = 0.0
    kern = np.nonzero(np.isin(g.kind, (W.K_ELEM, W.K_AUX, W.K_WU, W.K_GPU_OTHER)))[0]
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    words = torch.zeros((g.n, Wd), dtype=torch.int32, device=DEV)
    thr = torch.zeros(Wd * 32, dtype=torch.float32, device=DEV)
    thr[:V] = torch.from_numpy(dens.astype(np.float32)).to(DEV)
    shift = torch.arange(32, dtype=torch.int32, device=DEV)
    rows = max(1, (1 << 26) // (Wd * 32))

    def pack(bits):                          # [r][Wd * 32] truth values
        return torch.bitwise_left_shift(bits.view(-1, Wd, 32).to(torch.int32), shift).sum(2).to(torch.int32)

    def put(ids, w):
        at = torch.from_numpy(ids.astype(np.int64)).to(DEV)
        words[at] = w
        lo = g.launch_of[ids]
        words[torch.from_numpy(lo[lo >= 0].astype(np.int64)).to(DEV)] = w[torch.from_numpy(lo >= 0).to(DEV)]

    for s in range(0, kern.shape[0], rows):
        ids = kern[s:s + rows]
        put(ids, pack(torch.rand((ids.shape[0], Wd * 32), device=DEV, generator=gen) < thr))
    if case["model"] == "vdnn":
        copies = np.nonzero((g.kind == W.K_MEMCPY) & np.isin(g.op, (W.OP_OFFLOAD, W.OP_PREFETCH)))[0]
        none = torch.zeros(Wd * 32, dtype=torch.bool, device=DEV)
        none[5:V:5] = True                   # policy 0 of five (variant 0 stays as recorded)
        put(copies, pack(none.expand(copies.shape[0], -1).contiguous()))
    return words


def _edge_on(case):
    """uint64 [V] and the batches (v0, v1, mask) that share a schedule."""
    V = case["variants"]
    if case["model"] == "allreduce":
        per = V // 4
        ends = [0, per, 2 * per, 3 * per, V]
        on = np.concatenate([np.full(ends[i + 1] - ends[i], 1 | 1 << (1 + i), np.uint64) for i in range(4)])
        return on, [(ends[i], ends[i + 1], 1 | 1 << (1 + i)) for i in range(4)]
    if case["model"] == "vdnn":
        pol = np.arange(V) % 5
        return np.where(pol >= 2, 1 | 1 << np.maximum(pol - 1, 0), 1).astype(np.uint64), [(0, V, 0xF)]
    return np.ones(V, np.uint64), [(0, V, 1)]


def _inputs(case, seed):
    """(graph, DeviceInputs, push/pull flags, priorities)"""
    rng = np.random.default_rng(int(seed))
    g, rep, pp, prio = _graph(case, seed)

    def t(a):
        return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    scale = _scales(case, g, rep, rng)
    words = _removals(case, g, rng, seed)
    on, ranges = _edge_on(case)
    ten = dict(in_ptr=t(g.in_ptr.astype(np.int64)), in_src=t(g.in_src), edge_cls=t(g.edge_cls),
               thread_prev=t(g.thread_prev), thread_id=t(g.thread_id), dur=t(g.dur), gap=t(g.gap),
               node_cls=t(g.node_cls))
    batches = []
    for v0, v1, mask in ranges:
        if len(ranges) == 1:
            rm = words
        else:                                # the batch's own columns
            cols = torch.arange(v0, v1, device=DEV)
            bits = (words[:, cols // 32] >> (cols % 32).to(torch.int32)) & 1
            w2 = (v1 - v0 + 31) // 32
            pad = torch.zeros((g.n, w2 * 32), dtype=torch.int32, device=DEV)
            pad[:, :v1 - v0] = bits
            rm = torch.bitwise_left_shift(pad.view(g.n, w2, 32), torch.arange(32, dtype=torch.int32, device=DEV)).sum(2).to(torch.int32)
        batches.append((v0, v1, mask, t(scale[:, v0:v1]), rm.contiguous().view(torch.uint32), t(on[v0:v1])))
    return g, batch.DeviceInputs(g.n, g.n_threads, ten, batches, g.n_node_cls, case["variants"]), pp, prio


class _Handles:
    """Library handles that live as long as the state that keeps them."""

    def __init__(self):
        self.graph = None
        self.sched, self.var = [], []

    def __del__(self):
        if sys.is_finalizing():
            return
        for s in self.sched:
            B.dd_sched_free(s)
        for v in self.var:
            B.dd_variants_free(v)
        B.dd_graph_free(self.graph)


def prepare(case, seed):
    g, di, pp, prio = _inputs(case, seed)
    path, start = case["path"], case["start"]
    outs = []
    for v0, v1, *_ in di.batches:
        shape = (g.n, v1 - v0)
        outs.append((torch.empty(shape, dtype=torch.int64, device=DEV),
                     torch.empty(shape, dtype=torch.int64, device=DEV) if start and path != "breakdown" else None,
                     torch.empty(v1 - v0, dtype=torch.int64, device=DEV)))
    state = dict(path=path, di=di, outs=outs)
    if path == "step":
        return state
    h = state["handles"] = _Handles()
    if path == "policy":
        x = di.tensors
        h.graph = B.dd_graph_load_ex(di.n, di.n_threads, x["in_ptr"], x["in_src"], x["edge_cls"], x["thread_prev"],
                                     x["thread_id"], x["dur"], x["gap"], x["node_cls"], B.DD_LOAD_SHARED_THREADS)
        state["rule"] = B.DD_POLICY_PRIORITY if case["iters"] > 4 else B.DD_POLICY_EARLIEST
        state["pp"], state["prio"] = torch.from_numpy(pp).to(DEV), torch.from_numpy(prio).to(DEV)
        return state
    h.graph = batch.load_graph(di)
    h.sched = [B.dd_levelize(h.graph, mask, B.DD_PHASES)[0] for _, _, mask, *_ in di.batches]
    if path == "breakdown":
        state["role"] = torch.from_numpy(W.task_roles(g)).to(DEV)
        state["parts"] = []
        for (v0, v1, _m, scale, rm, on), sch, (fin, _s, ms) in zip(di.batches, h.sched, outs):
            var = B.dd_apply_transforms(h.graph, v1 - v0, di.n_cls, scale, rm, on)
            h.var.append(var)
            B.dd_simulate_batch(h.graph, sch, var, fin, None, ms)
            state["parts"].append(torch.empty((v1 - v0, 4), dtype=torch.int64, device=DEV))
    return state


# ---------------------------------------------------------------------------
# one pass
def run(state):
    path, di, outs = state["path"], state["di"], state["outs"]
    if path == "step":
        batch.simulate(di, outputs=outs)
        return outs
    h = state["handles"]
    if path == "sweep":
        for (v0, v1, _m, scale, rm, on), sch, (fin, st, ms) in zip(di.batches, h.sched, outs):
            var = B.dd_apply_transforms(h.graph, v1 - v0, di.n_cls, scale, rm, on)
            B.dd_simulate_batch(h.graph, sch, var, fin, st, ms)
            B.dd_variants_free(var)
        return outs
    if path == "policy":
        (_v0, _v1, _m, scale, rm, on), (fin, st, ms) = di.batches[0], outs[0]
        var = B.dd_apply_transforms(h.graph, di.n_variants, di.n_cls, scale, rm, on)
        B.dd_simulate_policy(h.graph, var, state["rule"], state["pp"], state["prio"], fin, st, ms)
        B.dd_variants_free(var)
        return outs
    for var, (fin, _s, ms), out in zip(h.var, outs, state["parts"]):
        B.dd_runtime_breakdown(h.graph, var, state["role"], fin, ms, out)
    return state["parts"]


# ---------------------------------------------------------------------------
def work(case):
    tasks, cross, roles, waits = (x * case["iters"] for x in SHAPE[case["model"]])
    V = case["variants"]
    classes = 30 * V * 8.0                   # scale ratios (classes of an ordinary trace)
    removed = tasks * V / 8.0
    if case["path"] == "breakdown":
        return {"bytes": classes + roles * V / 8.0 + waits * V * 16.0 + tasks * 5.0 + roles * 10.0 + V * 40.0, "flops": 0}
    finish = tasks * V * (16.0 if case["start"] else 8.0) + V * 8.0
    graph = tasks * 38.0 + cross * 5.0       # the trace's arrays, or the schedule made of them
    if case["path"] == "policy":             # reference counts and starts are state that stays on the chip
        return {"bytes": finish + classes + removed + graph, "flops": 0}
    gathers = cross * V * 8.0                # each parent on another thread: its finish read back
    return {"bytes": finish + gathers + classes + removed + graph, "flops": 0}


def tolerance(case):
    return "exact"


# ---------------------------------------------------------------------------
# Algorithm 1 in plain numpy, a row of variants at a time
def _host(di, i):
    v0, v1, mask, scale, rm, on = di.batches[i]
    x = {k: t.cpu().numpy() for k, t in di.tensors.items()}
    p, q = (scale.cpu().numpy().astype(np.int64)[:, :, k] for k in (0, 1))
    w = rm.view(torch.int32).cpu().numpy()
    cols = np.arange(v1 - v0)
    return x, p, q, (lambda u: ((w[u][cols // 32] >> (cols % 32)) & 1) != 0), on.cpu().numpy(), mask


def _simulate(di, i):
    x, p, q, removed, on, mask = _host(di, i)
    n, V = di.n, p.shape[1]
    fin, rel, beg = (np.zeros((n, V), np.int64) for _ in range(3))
    ms = np.zeros(V, np.int64)
    dst = np.repeat(np.arange(n), np.diff(x["in_ptr"]))
    used = (mask >> x["edge_cls"].astype(np.int64)) & 1 != 0
    src, dst, cls = x["in_src"][used], dst[used], x["edge_cls"][used]
    present = [(on >> np.uint64(k)) & np.uint64(1) != 0 for k in range(64)]
    prev = x["thread_prev"]
    parents = [[] for _ in range(n)]
    children = [[] for _ in range(n)]
    for s, d, k in zip(src.tolist(), dst.tolist(), cls.tolist()):
        parents[d].append((s, k))
        children[s].append(d)
    count = np.bincount(dst, minlength=n) + (prev >= 0)
    for u in np.nonzero(prev >= 0)[0].tolist():
        children[prev[u]].append(u)
    ready = np.nonzero(count == 0)[0].tolist()
    while ready:
        u = ready.pop()
        s = rel[prev[u]].copy() if prev[u] >= 0 else np.zeros(V, np.int64)
        for a, k in parents[u]:
            np.maximum(s, np.where(present[k], rel[a], 0), out=s)
        c, gone = x["node_cls"][u], removed(u)
        d = np.where(gone, 0, x["dur"][u] * p[c] // q[c])
        beg[u], fin[u] = s, s + d
        rel[u] = fin[u] + np.where(gone, 0, x["gap"][u])
        np.maximum(ms, np.where(gone, 0, fin[u]), out=ms)
        for a in children[u]:
            count[a] -= 1
            if count[a] == 0:
                ready.append(a)
    return fin, beg, rel, ms


def _policy(di, priority, pp, prio):
    x, p, q, removed, on, _mask = _host(di, 0)
    n, V = di.n, p.shape[1]
    fin, beg, ms = np.zeros((n, V), np.int64), np.zeros((n, V), np.int64), np.zeros(V, np.int64)
    gone = np.stack([removed(u) for u in range(n)])
    dst = np.repeat(np.arange(n), np.diff(x["in_ptr"])).tolist()
    for v in range(V):
        children, count = [[] for _ in range(n)], [0] * n
        for s, d, k in zip(x["in_src"].tolist(), dst, x["edge_cls"].tolist()):
            if int(on[v]) >> k & 1:
                children[s].append(d)
                count[d] += 1
        for u, a in enumerate(x["thread_prev"].tolist()):
            if a >= 0:
                children[a].append(u)
                count[u] += 1
        free, start = [0] * di.n_threads, [0] * n
        front = [u for u in range(n) if count[u] == 0]
        while front:
            best, at = None, None
            for u in sorted(front):
                t = max(free[x["thread_id"][u]], start[u])
                if best is None or t < at:
                    best, at = u, t
                elif priority and t == at and pp[u] and pp[best] and prio[u] > prio[best]:
                    best = u
            front.remove(best)
            c, off = x["node_cls"][best], gone[best, v]
            f = at + (0 if off else int(x["dur"][best]) * int(p[c, v]) // int(q[c, v]))
            r = f + (0 if off else int(x["gap"][best]))
            beg[best, v], fin[best, v], free[x["thread_id"][best]] = at, f, r
            ms[v] = max(ms[v], 0 if off else f)
            for a in children[best]:
                start[a] = max(start[a], r)
                count[a] -= 1
                if count[a] == 0:
                    front.append(a)
    return fin, beg, ms


def exact(case, seed):
    pairs = SHAPE[case["model"]][0] * case["iters"] * case["variants"]
    if pairs > (30_000 if case["path"] == "policy" else 60_000_000):
        return None
    g, di, pp, prio = _inputs(case, seed)
    if case["path"] == "policy":
        fin, beg, ms = _policy(di, case["iters"] > 4, pp, prio)
        return [(fin, beg if case["start"] else None, ms)]
    got = []
    for i in range(len(di.batches)):
        fin, beg, rel, ms = _simulate(di, i)
        if case["path"] != "breakdown":
            got.append((fin, beg if case["start"] else None, ms))
            continue
        x, p, q, removed, _on, _mask = _host(di, i)
        role, prev = W.task_roles(g), x["thread_prev"]
        kernels, blocked = np.zeros(ms.shape, np.int64), np.zeros(ms.shape, np.int64)
        for u in np.nonzero(role == 1)[0].tolist():
            kernels += fin[u] - beg[u]
        for u in np.nonzero(role == 2)[0].tolist():
            blocked += beg[u] - (rel[prev[u]] if prev[u] >= 0 else 0)
        got.append(np.stack([ms, ms - kernels, blocked, kernels - blocked], axis=1))
    return got
