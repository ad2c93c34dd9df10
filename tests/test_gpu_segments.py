"""GPU parity of the composer's segments and linked collectives, through the C ABI.

The sweep walks runs of compute and memcpy ops (segments, at most 32 ops, 64-record
chunks) and lets a collective be announced before the collective it follows on its
streams is done (links).  These graphs sit at the edges: runs of 1, 31, 32, 33, 64, 65
ops, runs broken by an op something else waits for, memcpy ops inside a run, a second
compute stream, comm ops without dependencies launching in the middle of a run, chains of
collectives of 3 members (member slots) and of 24 (counted arrivals), a stream that carries
two communicators (no link), several ranks per wavefront (streams without a slot), and
collectives on the compute streams.
Integers, so every start, finish, step and digest must equal the oracle's.
"""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from tests.test_gpu_parity import THREADS, assert_same, gpu_run
from tests.tinygraph import AG, AR, MEMCPY, P2P, RS, Builder, folded_link, shared_streams
from workloads import scenarios

pytestmark = pytest.mark.gpu
RUNS = (1, 2, 7, 31, 32, 33, 64, 65)


@pytest.fixture(scope="module")
def E():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2412_12487_amd as E
    E.lib()
    return E


def spmd_graph(seed, ranks=24, steps=10, buckets=6, shared=False):
    """Every rank runs the same program: per step a run of compute ops, then sometimes a
    pairwise exchange, a bucket reduction over ranks r, r + 8, r + 16 (stream 2) or over all
    ranks (stream 1), or a send/recv to rank r +- 8; at the end one op per bucket waits for it.
    shared: the reductions run on the compute streams 0 and 6 instead."""
    rng = np.random.default_rng(seed)
    b = Builder(ranks, gpus_per_node=4)
    plan = []
    for _ in range(steps):
        plan.append((int(rng.choice(RUNS)), rng.choice(["none", "bucket", "bucket", "all", "p2p", "free", "tp"]),
                     int(rng.integers(0, 3)), bool(rng.random() < 0.3)))
    plan += [(1, "bucket", 0, False)] * buckets + [(2, "all", 0, False)] * 2
    colls = []
    for _, kind, _, _ in plan:
        size = int(rng.integers(0, 48 << 20))
        if kind == "bucket" or kind == "free":
            t = int(rng.choice([AR, RS, AG]))
            colls.append([b.collective(t, size) for _ in range(8)])
        elif kind == "all":
            colls.append([b.collective(AR, size)])
        elif kind == "tp":
            colls.append([b.collective(AR, size) for _ in range(ranks // 4)])
        elif kind == "p2p":
            colls.append([b.collective(P2P, size) for _ in range(8)])
        else:
            colls.append([])
    on = lambda stream: {1: 6, 2: 0, 7: 0}[stream] if shared else stream
    for r in range(ranks):
        tail, waits, buckets_of = -1, [], []
        for (run, kind, side, copy), ids in zip(plan, colls):
            for k in range(run):
                preds = waits if k == 0 else [tail] if rng.random() < 0.5 else []
                if copy and k == run // 2:
                    tail = b.op(r, kind=MEMCPY, dur=int(rng.integers(0, 9000)), preds=preds)
                else:
                    tail = b.compute(r, int(rng.integers(0, 60_000)), cls=int(rng.integers(0, 8)), preds=preds)
                waits = []
                if side == 1 and k == 3:      # a second compute stream waits for the middle of the run
                    b.compute(r, int(rng.integers(0, 40_000)), stream=6, cls=k, preds=[tail])
                if side == 2 and k == 5:
                    b.op(r, stream=5, kind=MEMCPY, dur=700)
            if kind == "bucket":
                buckets_of.append(b.comm(r, ids[r % 8], stream=on(2), preds=[tail]))
            elif kind == "free":              # no dependency but its stream: launches whenever that is free
                b.comm(r, ids[r % 8], stream=on(2))
            elif kind == "all":
                buckets_of.append(b.comm(r, ids[0], stream=on(1 if side else 2), preds=[tail]))
            elif kind == "tp":
                waits = [b.comm(r, ids[r // 4], stream=on(7), preds=[tail])]
            elif kind == "p2p" and r < 16:
                waits = [b.comm(r, ids[r % 8], stream=3 if r < 8 else 4, preds=[tail])] if r >= 8 else []
                if r < 8:
                    b.comm(r, ids[r % 8], stream=3, preds=[tail])
        for c in buckets_of:
            tail = b.compute(r, int(rng.integers(0, 5_000)), cls=6, preds=[c])
    return b.graph()


@pytest.mark.parametrize("seed", range(8))
@pytest.mark.parametrize("rpw", [0, 3])
def test_segments_and_links(E, seed, rpw):
    g = spmd_graph(seed)
    n = [1, 64, 70, 130][seed % 4]
    sc = scenarios.draw(n, np.random.default_rng(seed), bw_inter=(5_000, 400_000), bw_intra=(20_000, 400_000),
                        alpha=(0, 20_000), ar_algo_random=True, slowdown=(65536, 150_000),
                        jitter=(9000, seed) if seed % 2 else None)
    G = E.Graph(g, 0, ranks_per_walker=rpw)
    try:
        for R in (0, 1, 2):
            assert_same(gpu_run(E, g, sc, R, graph=G), oracle.run(g, sc, R, threads=THREADS))
        d, n = E.scenarios_to_device(sc)
        steps = G.compose(d, n, 2, timelines=False)["step"].cpu().numpy()      # no timelines: same steps
        np.testing.assert_array_equal(steps, oracle.run(g, sc, 2, threads=THREADS, timelines=False)["step"])
        for kw in ({"until_stable": True}, {"prorate": True}, {"until_stable": True, "prorate": True}):
            ref = oracle.run(g, sc, 5, threads=THREADS, **kw)
            out = G.compose(d, n, 5, timelines=True, digest=True, refinements=True, **kw)
            assert_same({"step": out["step"].cpu().numpy(), "digest": out["digest"].cpu().numpy().view(np.uint64),
                         "start": out["start"].cpu().numpy(), "finish": out["finish"].cpu().numpy()}, ref)
            np.testing.assert_array_equal(out["refinements"].cpu().numpy(), ref["refinements"])
    finally:
        G.close()


@pytest.mark.parametrize("rpw", [0, 3])
@pytest.mark.parametrize("order", ["uxv", "xuv", "uvx"])
def test_collectives_on_the_compute_stream_beside_a_folded_one(E, order, rpw):
    """A comm op of the compute stream, linked or not, and one of another stream are resolved
    before the same segment: neither's finish may stand in for the other's."""
    g = folded_link(order)
    sc = scenarios.draw(70, np.random.default_rng(1), bw_inter=(5_000, 400_000), slowdown=(65536, 150_000))
    with E.Graph(g, 0, ranks_per_walker=rpw) as G:
        for R in (0, 1):
            assert_same(gpu_run(E, g, sc, R, graph=G), oracle.run(g, sc, R, threads=THREADS))


@pytest.mark.parametrize("rpw", [0, 3])
@pytest.mark.parametrize("seed", range(12))
def test_collectives_on_compute_streams(E, seed, rpw):
    rng = np.random.default_rng(seed)
    g = spmd_graph(seed, shared=True) if seed < 4 else shared_streams(rng)
    sc = scenarios.draw([1, 64, 70, 130][seed % 4], rng, bw_inter=(5_000, 400_000), bw_intra=(20_000, 400_000),
                        alpha=(0, 20_000), ar_algo_random=True, slowdown=(65536, 150_000),
                        jitter=(9000, seed) if seed % 2 else None)
    with E.Graph(g, 0, ranks_per_walker=rpw) as G:
        for R in (0, 2):
            assert_same(gpu_run(E, g, sc, R, graph=G), oracle.run(g, sc, R, threads=THREADS))


@pytest.mark.parametrize("seed,rpw,cap", [(0, 0, 0), (1, 0, 0), (3, 0, 7), (4, 3, 0), (5, 0, 0)])
def test_unrefined_timelines_from_the_sweep_of_the_ops(E, seed, rpw, cap):
    """From 48,000 evaluations per level and rank of a walker on (of one launch) the sweep walks the
    ops themselves: just below that line, at it and above, ragged tiles, base durations above
    2^32 ns, launches of a few tiles (cap), the allocation-free entry point, one output alone and
    no timelines."""
    import ctypes
    import torch
    rng = np.random.default_rng(seed)
    g = shared_streams(np.random.default_rng(0)) if seed == 5 else spmd_graph(seed, steps=2, buckets=1, shared=seed == 4)
    if seed == 1:
        wide = (np.arange(len(g["op_dur"])) % 11 == 0) & (g["op_kind"] == 0)
        g["op_dur"][wide] += 1 << 33
    with E.Graph(g, 0, ranks_per_walker=rpw) as G:
        line = -(-48_000 * G.n_levels * max(rpw, 1) // G.n_ops)
        for n in (line - 1, line, line + 70):
            n = n * 3 if cap else n
            sc = scenarios.draw(n, rng, bw_inter=(5_000, 400_000), alpha=(0, 20_000), ar_algo_random=True,
                                jitter=(9000, seed) if seed != 3 else None)
            ref = oracle.run(g, sc, 0, threads=THREADS)
            G.set_launch_tiles(-(-n // 64) // 3 if cap else 0)
            d, n = E.scenarios_to_device(sc)
            out = {k: torch.full((G.n_ops, n) if k != "step" else (n,), -1, dtype=torch.int64, device="cuda:0")
                   for k in ("start", "finish", "step")}
            G.compose(d, n, 0, out=out)
            outs = [out]
            if seed == 0:
                outs.append(G.compose_static(d, n, 0, {k: torch.full_like(v, -1) for k, v in out.items()}))
                alone = {k: torch.full_like(out[k], -1) for k in ("start", "finish")}     # one output each
                ptr = lambda t: ctypes.c_void_p(t.data_ptr())
                for k in alone:
                    rc = E.lib().echo_compose_batch(G.handle, ptr(d), n, 0, ptr(alone[k]) if k == "start" else None,
                                                    ptr(alone[k]) if k == "finish" else None, ptr(out["step"]), None,
                                                    ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
                    assert rc == E.ECHO_OK
                outs.append({"step": out["step"], **alone})
            for o in outs:
                np.testing.assert_array_equal(o["step"].cpu().numpy(), ref["step"])
                np.testing.assert_array_equal(o["start"].cpu().numpy().T, ref["start"])
                np.testing.assert_array_equal(o["finish"].cpu().numpy().T, ref["finish"])
            np.testing.assert_array_equal(G.compose(d, n, 0, timelines=False)["step"].cpu().numpy(), ref["step"])


def test_sweep_of_the_ops_and_direct_costs_in_a_hip_graph(E):
    """An unrefined compose on the sweep of the ops (three workgroups: a cooperative launch) and a
    small echo_cc_cost, captured and replayed with eager work between the replays."""
    import ctypes
    import torch
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    g = spmd_graph(0, steps=2, buckets=1)
    with E.Graph(g, 0) as G:
        n = -(-48_000 * G.n_levels // G.n_ops)
        sc = scenarios.draw(n, np.random.default_rng(5), bw_inter=(5_000, 400_000), jitter=(9000, 5))
        d, n = E.scenarios_to_device(sc)
        out = {k: torch.full((G.n_ops, n) if k != "step" else (n,), -1, dtype=torch.int64, device="cuda:0")
               for k in ("start", "finish", "step")}
        cost = torch.full((G.n_colls, n), -1, dtype=torch.int64, device="cuda:0")

        def calls():
            G.compose(d, n, 0, out=out, check=False)
            rc = E.lib().echo_cc_cost(G.handle, ptr(d), n, ptr(cost),
                                      ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
            assert rc == E.ECHO_OK

        torch.cuda.synchronize()
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            calls()                                # sizes the workspace
        torch.cuda.synchronize()
        ref = oracle.run(g, sc, 0, threads=THREADS, costs=True)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            calls()
        for _ in range(3):
            for v in (*out.values(), cost):
                v.fill_(-1)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            np.testing.assert_array_equal(out["step"].cpu().numpy(), ref["step"])
            np.testing.assert_array_equal(out["start"].cpu().numpy().T, ref["start"])
            np.testing.assert_array_equal(out["finish"].cpu().numpy().T, ref["finish"])
            np.testing.assert_array_equal(cost.cpu().numpy().T, ref["cost"])
        G.sync_status()
        del graph


def test_digest_alone_and_one_output_alone(E):
    """Digest without timelines, and start or finish alone through the C ABI."""
    import ctypes
    import torch
    g = spmd_graph(3)
    sc = scenarios.draw(70, np.random.default_rng(3), slowdown=(65536, 150_000), jitter=(9000, 3))
    ref = oracle.run(g, sc, 1, threads=THREADS)
    with E.Graph(g, 0) as G:
        d, n = E.scenarios_to_device(sc)
        out = G.compose(d, n, 1, timelines=False, digest=True)
        np.testing.assert_array_equal(out["digest"].cpu().numpy().view(np.uint64), ref["digest"])
        none, ptr = ctypes.c_void_p(None), lambda t: ctypes.c_void_p(t.data_ptr())
        for key in ("start", "finish"):
            buf = torch.full((G.n_ops, n), -1, dtype=torch.int64, device="cuda:0")
            step = torch.empty(n, dtype=torch.int64, device="cuda:0")
            rc = E.lib().echo_compose_batch(G.handle, ptr(d), n, 1, ptr(buf) if key == "start" else none,
                                            ptr(buf) if key == "finish" else none, ptr(step), none,
                                            ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
            assert rc == E.ECHO_OK
            G.sync_status()
            np.testing.assert_array_equal(buf.cpu().numpy().T, ref[key])
