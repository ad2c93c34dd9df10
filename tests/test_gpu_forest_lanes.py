"""GPU parity of the tree ensemble where only some scenarios of a tile overlap an op: the
scenarios share their ensemble features (one walk of the trees for the wavefront, one tree per
lane), and the lanes that overlap nothing hold trees that the others need."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from tests.test_gpu_parity import THREADS, assert_same
from tests.tinygraph import AG, P2P, Builder
from workloads import scenarios, slowdown_forest

pytestmark = pytest.mark.gpu


def two_ranks():
    """A send and an all-gather whose ends move with alpha over the compute ops beside them: op k
    is overlapped in the scenarios whose alpha reaches it."""
    b = Builder(2)
    p2p, ag = b.collective(P2P, 1 << 10), b.collective(AG, 1 << 20)
    for r in range(2):
        a = b.compute(r, 1000)
        b.comm(r, p2p, stream=3, preds=[a])
        b.comm(r, ag, stream=4, preds=[a])
        for k in range(12):
            b.compute(r, 2000 + 100 * k, cls=k % 8)
    return b.graph()


@pytest.mark.parametrize("trees", [5, 64, 128])
@pytest.mark.parametrize("n", [64, 70])
def test_lanes_without_overlap_still_walk_their_trees(trees, n):
    """5 and 64 trees are held in LDS, 128 are walked from device memory."""
    import paper_2412_12487_amd as E
    g, fo = two_ranks(), slowdown_forest.synthetic_forest(0, n_trees=trees)
    assert (len(fo["nodes"]) + len(fo["roots"]) <= 12 * 1024) == (trees <= 64)
    sc = scenarios.draw(n, np.random.default_rng(1))
    sc["alpha_ns"] = (np.arange(n, dtype=np.int64) * 7919 % n) * 400
    with E.Graph(g, 0) as G:
        G.set_forest(fo)
        d, n = E.scenarios_to_device(sc)
        for prorate in (False, True):
            ref = oracle.run(g, sc, 2, threads=THREADS, prorate=prorate, forest=fo)
            out = G.compose(d, n, 2, digest=True, forest=True, prorate=prorate)
            assert_same({"step": out["step"].cpu().numpy(), "digest": out["digest"].cpu().numpy().view(np.uint64),
                         "start": out["start"].cpu().numpy(), "finish": out["finish"].cpu().numpy()}, ref)
