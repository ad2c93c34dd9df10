"""The loader's walk lists, segments and overlap ranges, composed on the CPU by the host stub's
model of the kernels (tests/sanitize/composer_model.h) and compared with the oracle: every
start, finish, step, digest and refinement count.  Runs only inside the sanitizer run of
tests/test_sanitized_host.py."""
from __future__ import annotations

import ctypes
import os

import numpy as np
import pytest

import oracle
from tests import tinygraph
from workloads import configs, scenarios

pytestmark = pytest.mark.skipif(not os.environ.get("ECHO_HOST_STUB"),
                                reason="needs the sanitizer build linked with the HIP host stub")


@pytest.fixture(scope="module")
def E():
    import paper_2412_12487_amd as E
    E.lib().echo_stub_set_costs.argtypes = [ctypes.c_void_p]
    yield E
    E.lib().echo_stub_set_costs(None)


def check(E, g, sc, R, rpw=0, until_stable=False, prorate=False, digest=True):
    from paper_2412_12487_amd.echo import _Validator
    n = len(sc["alpha_ns"])
    ref = oracle.run(g, sc, R, costs=True, until_stable=until_stable, prorate=prorate)
    cost, rec = np.ascontiguousarray(ref["cost"].T), E.pack_scenarios(sc)
    E.lib().echo_stub_set_costs(cost.ctypes.data)
    with E.Graph(g, 0, ranks_per_walker=rpw) as G:
        out = {k: np.full((G.n_ops, n), -1, np.int64) for k in ("start", "finish")}
        out.update(step=np.zeros(n, np.int64), digest=np.zeros(n, np.uint64), refinements=np.zeros(n, np.int32))
        ptr = lambda a: ctypes.c_void_p(a.ctypes.data)
        if not digest:
            del out["digest"]
        opts = _Validator(R, int(until_stable), int(prorate), 0)
        rc = E.lib().echo_compose_validated(G.handle, ptr(rec), n, ctypes.byref(opts),
                                            *(ptr(out[k]) if k in out else None
                                              for k in ("start", "finish", "step", "digest", "refinements")), None)
        assert rc == E.ECHO_OK, E.lib().echo_last_error()
    for k, got in out.items():
        np.testing.assert_array_equal(got.T if got.ndim == 2 else got, ref[k], err_msg=k)


@pytest.mark.parametrize("order", ["uxv", "xuv", "uvx"])
def test_collectives_on_the_compute_stream_beside_a_folded_one(E, order):
    """Neither may x's finish, folded into the compute stream's slot, enter v (linked to u), nor
    may v's finish replace it there."""
    sc = scenarios.draw(3, np.random.default_rng(1), slowdown=(65536, 150_000))
    for R in (0, 1):
        check(E, tinygraph.folded_link(order), sc, R)


@pytest.mark.parametrize("seed", range(60))
def test_random_graphs_with_shared_streams(E, seed):
    rng = np.random.default_rng(seed)
    g = tinygraph.shared_streams(rng)
    sc = scenarios.draw(70 if seed % 20 == 0 else 2, rng, bw_inter=(5_000, 400_000), bw_intra=(20_000, 400_000),
                        alpha=(0, 20_000), ar_algo_random=True, slowdown=(65536, 150_000),
                        jitter=(9000, seed) if seed % 2 else None)
    check(E, g, sc, seed % 3, rpw=seed % 5)
    check(E, g, sc, 2, prorate=True)
    check(E, g, sc, 5, rpw=seed % 2, until_stable=True, prorate=seed % 4 == 1)


IN_NONE, IN_OPS = 0, 4        # inputs of a sweep (echo_internal.h)


@pytest.mark.parametrize("seed,rpw", [(0, 0), (3, 0), (8, 0), (2, 1), (3, 3), (0, 5)])
def test_sweep_of_the_ops_from_its_line_on(E, seed, rpw):
    """Unrefined timelines come from one sweep of the ops from 48,000 evaluations per level and rank
    of a walker on, and from segments below: the same times on both sides of the line."""
    rng = np.random.default_rng(seed)
    g = tinygraph.shared_streams(rng)
    with E.Graph(g, 0) as G:
        line = -(-48_000 * G.n_levels * max(rpw, 1) // G.n_ops)
    for n, used in ((line - 1, IN_NONE), (line, IN_OPS)):
        sc = scenarios.draw(n, rng, bw_inter=(5_000, 400_000), alpha=(0, 20_000), jitter=(9000, seed) if seed % 2 else None)
        check(E, g, sc, 0, rpw=rpw, digest=False)
        assert E.lib().echo_stub_sweep_in() == used
        check(E, g, sc, 0, rpw=rpw)                       # a digest keeps the segments
        assert E.lib().echo_stub_sweep_in() == IN_NONE


def test_gpt_graph(E):
    sc = scenarios.draw(2, np.random.default_rng(3), bw_inter=configs.BW_RANGE, alpha=configs.ALPHA_RANGE)
    check(E, configs.graph(1), sc, 1)
