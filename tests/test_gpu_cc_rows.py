"""GPU parity of echo_cc_cost.  Small calls cost every collective by itself; where copies replace
enough evaluations every collective's row is its cost class's, copied two scenarios at a time
where the rows are 16-byte aligned and one at a time elsewhere."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest

import oracle
from tests.test_gpu_segments import spmd_graph
from tests.tinygraph import AG, AR, RS, Builder
from workloads import scenarios

pytestmark = pytest.mark.gpu


def many_collectives():
    """8000 collectives of 19 classes on two ranks."""
    b = Builder(2)
    ids = [b.collective((AR, AG, RS)[k % 3], 1000 + 997 * (k % 19) ** 4) for k in range(8000)]
    for r in range(2):
        for c in ids:
            b.comm(r, c)
    return b.graph()


# up to about 200 scenarios x 4000 copied rows every collective is costed by itself
@pytest.mark.parametrize("graph,n", [("few", n) for n in (1, 2, 63, 64, 130, 257)] +
                         [("many", n) for n in (63, 128, 193, 257)])
@pytest.mark.parametrize("shift", [0, 1])
def test_every_collective_has_its_class_cost(graph, n, shift):
    """shift: the output starts 8 bytes past a 16-byte boundary."""
    import torch
    import paper_2412_12487_amd as E
    g = spmd_graph(2) if graph == "few" else many_collectives()
    sc = scenarios.draw(n, np.random.default_rng(n), bw_inter=(5_000, 400_000), bw_intra=(20_000, 400_000),
                        alpha=(0, 20_000), ar_algo_random=True)
    sc["cc_model"] = (np.arange(n) % 2).astype(np.uint8)
    ref = oracle.run(g, sc, 0, timelines=False, costs=True)["cost"].T
    with E.Graph(g, 0) as G:
        d, n = E.scenarios_to_device(sc)
        np.testing.assert_array_equal(G.cc_cost(d, n).cpu().numpy(), ref)
        out = torch.full((G.n_colls * n + 2,), -7, dtype=torch.int64, device="cuda:0")
        assert out.data_ptr() % 16 == 0
        assert E.lib().echo_cc_cost(G.handle, ctypes.c_void_p(d.data_ptr()), n,
                                    ctypes.c_void_p(out.data_ptr() + 8 * shift),
                                    ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == E.ECHO_OK
        G.sync_status()
        got = out.cpu().numpy()
        np.testing.assert_array_equal(got[shift:shift + ref.size].reshape(ref.shape), ref)
        assert (got[:shift] == -7).all() and (got[shift + ref.size:] == -7).all()
