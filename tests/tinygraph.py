"""Hand-built execution graphs for the tests (same array layout as workloads.gpt1f1b)."""
from __future__ import annotations

import numpy as np

COMPUTE, COMM, MEMCPY = 0, 1, 2
AR, AG, RS, P2P = 0, 1, 2, 3


class Builder:
    """Append ops in rank-major program order; collectives are declared first."""

    def __init__(self, n_ranks, gpus_per_node=8):
        self.n_ranks, self.gpn = n_ranks, gpus_per_node
        self.rank, self.stream, self.kind, self.cls, self.dur, self.coll, self.preds = ([] for _ in range(7))
        self.ctype, self.cbytes = [], []

    def collective(self, ctype, nbytes):
        self.ctype.append(ctype)
        self.cbytes.append(nbytes)
        return len(self.ctype) - 1

    def op(self, rank, *, stream=0, kind=COMPUTE, cls=0, dur=0, coll=-1, preds=()):
        self.rank.append(rank)
        self.stream.append(stream)
        self.kind.append(kind)
        self.cls.append(cls)
        self.dur.append(dur)
        self.coll.append(coll)
        self.preds.append(list(preds))
        return len(self.rank) - 1

    def compute(self, rank, dur, *, stream=0, cls=0, preds=()):
        return self.op(rank, stream=stream, kind=COMPUTE, cls=cls, dur=dur, preds=preds)

    def comm(self, rank, coll, *, stream=1, preds=()):
        return self.op(rank, stream=stream, kind=COMM, cls=7, coll=coll, preds=preds)

    def graph(self):
        pc = [len(p) for p in self.preds]
        off = np.zeros(len(pc) + 1, np.int64)
        np.cumsum(pc, out=off[1:])
        return {
            "op_rank": np.array(self.rank, np.int32),
            "op_stream": np.array(self.stream, np.uint8),
            "op_kind": np.array(self.kind, np.uint8),
            "op_class": np.array(self.cls, np.uint8),
            "op_dur": np.array(self.dur, np.int64),
            "op_coll": np.array(self.coll, np.int64),
            "pred_off": off,
            "pred_idx": np.array([u for p in self.preds for u in p], np.int32),
            "coll_type": np.array(self.ctype, np.uint8),
            "coll_bytes": np.array(self.cbytes, np.int64),
            "n_ranks": self.n_ranks,
            "gpus_per_node": self.gpn,
        }


def pipeline_1f1b(P, m, tf, tb, gpus_per_node=8):
    """Pure 1F1B pipeline: one forward and one backward kernel per (stage,
    microbatch), activations/gradients exchanged by P2P pairs (zero bytes)."""
    b = Builder(P, gpus_per_node)
    ids = {}

    def pid(kind, boundary, mb):
        key = (kind, boundary, mb)
        if key not in ids:
            ids[key] = b.collective(P2P, 0)
        return ids[key]

    for p in range(P):           # declare collectives in a fixed order first
        for k in range(m):
            if p < P - 1:
                pid("f", p, k)
                pid("b", p, k)
    for p in range(P):
        last = [None]
        wait = []

        def compute(d):
            nonlocal wait
            v = b.compute(p, d, preds=wait)
            wait = []
            last[0] = v

        def comm(c, stream, blocking):
            v = b.comm(p, c, stream=stream, preds=[last[0]] if last[0] is not None else [])
            if blocking:
                wait.append(v)

        W = min(P - p - 1, m)
        R = m - W
        k = j = 0
        for _ in range(W):
            if p > 0:
                comm(pid("f", p - 1, k), 4, True)
            compute(tf)
            if p < P - 1:
                comm(pid("f", p, k), 3, False)
            k += 1
        if R > 0 and p > 0:
            comm(pid("f", p - 1, k), 4, True)
        for i in range(R):
            compute(tf)
            if p < P - 1:
                comm(pid("f", p, k), 3, False)
                comm(pid("b", p, j), 4, True)
            k += 1
            compute(tb)
            if p > 0:
                comm(pid("b", p - 1, j), 3, False)
                if i < R - 1:
                    comm(pid("f", p - 1, k), 4, True)
            j += 1
        for _ in range(W):
            comm(pid("b", p, j), 4, True)
            compute(tb)
            if p > 0:
                comm(pid("b", p - 1, j), 3, False)
            j += 1
    return b.graph()


def folded_link(order):
    """16 ranks; on the compute stream of each the all-reduces u, then v, both over {r, r + 8}, and
    on stream 1 a long one, x; the last compute op waits for v (its stream) and x.  order: the
    program order of the three, as a string; where x comes before u, the latest it may be
    resolved is still that op."""
    b = Builder(16, gpus_per_node=4)
    ids = {k: [b.collective(AR, size) for _ in range(8)] for k, size in (("u", 1 << 20), ("v", 1 << 20), ("x", 512 << 20))}
    for r in range(16):
        a = b.compute(r, 1000)
        b.compute(r, 2000, cls=1)
        op = {k: b.comm(r, ids[k][r % 8], stream=1 if k == "x" else 0, preds=[a]) for k in order}
        b.compute(r, 500, cls=2, preds=[op["x"]])
    return b.graph()


def shared_streams(rng):
    """Random ranks running one program of collectives in one order (so nothing deadlocks): pairs
    over workgroups, all ranks, groups of four, random sets; comm ops, compute and memcpy ops
    share streams 0, 1 and 6, with random dependencies."""
    ranks = int(rng.integers(2, 28))
    b = Builder(ranks, gpus_per_node=4)
    plan, own = [], bool(rng.random() < 0.3)      # own: comm ops on streams of their own
    for _ in range(int(rng.integers(2, 16))):
        kind, stream = int(rng.integers(0, 4)), int(rng.integers(1, 4) if own else rng.integers(0, 3))
        groups = [[r, r + 8] for r in range(max(0, min(8, ranks - 8)))] if kind == 0 else \
            [list(range(ranks))] if kind == 1 else \
            [list(range(i, min(i + 4, ranks))) for i in range(0, ranks, 4)] if kind == 2 else \
            [sorted(rng.choice(ranks, size=int(rng.integers(1, ranks + 1)), replace=False).tolist())]
        size = int(rng.integers(0, 64 << 20))
        plan += [(b.collective(int(rng.choice([AR, AG, RS])), size), set(m), stream) for m in groups]
    for r in range(ranks):
        ids = []

        def some(n, p):
            return [u for u in ids[-n:] if rng.random() < p]

        def work(streams, p):
            copy = rng.random() < 0.15
            ids.append(b.op(r, stream=int(rng.choice(streams)), kind=MEMCPY if copy else COMPUTE,
                            cls=int(rng.integers(0, 8)), dur=int(rng.integers(0, 60_000)), preds=some(6, p)))

        for c, members, stream in plan:
            if r not in members:
                continue
            for _ in range(int(rng.integers(0, 4))):
                work([0, 0, 0, 6, 1], 0.2)
            ids.append(b.comm(r, c, stream=stream, preds=some(4, 0.3)))
        for _ in range(3):
            work([0, 6], 0.4)
    return b.graph()
