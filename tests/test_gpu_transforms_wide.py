"""dd_apply_transforms with so many variants that several blocks fold the
edge-class masks: a class that one variant alone switches on, or off, is
noticed wherever that variant is (a simulation against a schedule without the
class is refused), and the results are the oracle's."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2006_03318_amd import batch as BT
from paper_2006_03318_amd import binding as B
from paper_2006_03318_amd import workloads as W
from tests import helpers as H
from tests.gpu_common import assert_equal_arrays, gpu_run, require_gpu, say

pytestmark = pytest.mark.gpu


def _graph():
    return H.graph(2, [0, 0, 1, 1], [(0, 3), (2, 1)], [5, 7, 11, 13], [1, 0, 2, 0], edge_cls=[0, 1], n_edge_cls=2)


@pytest.mark.parametrize("V", [1, 2047, 2048, 2049, 4097, 131_072, 131_073, 300_000])
@pytest.mark.parametrize("host", [False, True])
def test_masks_of_many_variants(V, host):
    import torch
    require_gpu()
    g = _graph()
    gh = BT.load_graph(BT.to_device(g, H.variants(g, V=1)))
    sch, _ = B.dd_levelize(gh, 1, B.DD_PHASES)            # without class 1
    fin = torch.empty((g.n, V), dtype=torch.int64, device="cuda")
    ms = torch.empty(V, dtype=torch.int64, device="cuda")
    for at in sorted({0, V // 3, max(0, V - 257), V - 1}):
        on = np.ones(V, np.uint64)
        say("masks V=%d host=%d at=%d" % (V, host, at))
        for odd, want in ((1, B.DD_OK), (3, B.DD_EMISMATCH)):
            on[at] = odd
            var = B.dd_apply_transforms(gh, V, 1, None, None, on if host else torch.from_numpy(on).cuda())
            rc = B.lib().dd_simulate_batch(gh, sch, var, fin.data_ptr(), None, ms.data_ptr(), None)
            torch.cuda.synchronize()
            B.dd_variants_free(var)
            assert rc == want, B.dd_last_error()
    B.dd_sched_free(sch)
    B.dd_graph_free(gh)


def test_results_with_many_variants():
    require_gpu()
    g = _graph()
    V = 5000
    rng = np.random.default_rng(3)
    vs = W.VariantSet(V, rng.integers(1, 4, (1, V, 2)).astype(np.int32), W.pack_bits(rng.random((g.n, V)) < 0.2),
                      rng.integers(0, 4, (V, 1)).astype(np.uint64), [(0, V, 3)])
    S, F, M = gpu_run(g, vs)
    oS, oF, oM, _ = O.run(g, vs)
    assert_equal_arrays("makespan", M, oM)
    assert_equal_arrays("finish", F, oF)
    assert_equal_arrays("start", S, oS)
