"""Runtime breakdown at the edges of its workgroups, bit-exact against the
oracle: chunks of 256 and 512 tasks, blocks of 128 variants, removal rows
that end inside a block, more classes than the sort has buckets, and the
integer form of the scaled durations."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2006_03318_amd import workloads as W
from tests.gpu_common import assert_equal_arrays, require_gpu, say
from tests.test_gpu_breakdown import gpu_breakdown

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,V,classes,big", [
    (1, 1, 1, False), (255, 127, 3, False), (256, 128, 1, False), (257, 129, 3, False),
    (2049, 31, 1500, False), (70_000, 257, 40, False), (300_001, 65, 2100, False),
    (3000, 130, 5, True)])
def test_breakdown_edges(n, V, classes, big):
    require_gpu()
    rng = np.random.default_rng(191_000 + n + V)
    g = W.random_graph_sparse(rng, n, 3, mean_in=0.2, window=100, n_node_cls=classes, run_len=50,
                              max_dur=2**44 if big else 10**5)
    vs = W.random_variants(rng, g, min(V, 40), p_remove=0.3)
    if V > 40:                       # the same variants again, in other places of the rows
        at = rng.integers(0, 40, V)
        bits = W.unpack_bits(vs.remove_bits, 40)[:, at]
        vs = W.VariantSet(V, np.ascontiguousarray(vs.scale[:, at]), W.pack_bits(bits),
                          np.ascontiguousarray(vs.edge_on[at]), [(0, V, vs.batches[0][2])])
    role = rng.integers(0, 4, size=g.n).astype(np.uint8)
    if n > 200_000:
        role[role == 2] = 1          # (a handful of waiting calls, as in a trace)
        role[:: 1000] = 2
    say("breakdown edges n=%d V=%d classes=%d big=%d" % (n, V, classes, big))
    assert_equal_arrays("breakdown", gpu_breakdown(g, vs, role), O.breakdown(g, vs, role))


@pytest.mark.parametrize("n,V", [(1, 129), (2, 1), (255, 128), (513, 130), (2048, 257)])
def test_every_task_waits(n, V):
    """Waiting calls alone, an odd number and an even one in a chunk: the two
    threads of a variant take them in turn."""
    require_gpu()
    rng = np.random.default_rng(192_000 + n + V)
    g = W.random_graph_sparse(rng, n, 3, mean_in=0.4, window=100, n_node_cls=4, run_len=7)
    vs = W.random_variants(rng, g, V, p_remove=0.3)
    role = np.full(n, 2, np.uint8)
    say("breakdown of waiting calls n=%d V=%d" % (n, V))
    assert_equal_arrays("breakdown", gpu_breakdown(g, vs, role), O.breakdown(g, vs, role))
