"""Performance cases of the timeline composer, through the binding's public entry points.

A case is one graph recipe (a synthetic GPT training job, `workloads.gpt1f1b`), one recipe of
what-if scenarios and one call: `Graph.compose` with its options, `Graph.compose_static` or
`Graph.cc_cost`.  The graph and the scenarios are loaded before the call, as a program that
composes more than one batch does; durations, jitter and scenario knobs come from the seed.

Keys of a case (all plain values):
    call        "compose", "static" (the allocation-free compose) or "cc_cost"
    layers, hidden, seq, tp, pp, dp, mb, distopt    the job (`gpt1f1b.gpt_graph`)
    replica     compose one data-parallel replica of the job instead of every rank
    n           scenarios
    jitter      every duration jittered by +-10 %
    vary        which knobs differ between scenarios: "none", "net" (bandwidths, alpha),
                "all" (also ring/tree and the slowdown tables)
    cc          collective cost model: "echo", "tables" (CC parameter tables) or "mixed"
                (the alpha-beta baseline and tables side by side)
    refine, stable, prorate, forest                 validator options
    timelines, digest, check                        outputs, and whether the call waits and checks
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2412_12487_amd as E
from workloads import configs, gpt1f1b, scenarios, slowdown_forest

DEFAULTS = dict(call="compose", layers=2, hidden=1024, seq=512, tp=2, pp=2, dp=2, mb=4, distopt=False, replica=False,
                n=1, jitter=False, vary="all", cc="echo", refine=1, stable=False, prorate=False, forest=False,
                timelines=True, digest=False, check=False)
GPT70B = dict(layers=80, hidden=8192, seq=2048)
GPT175B = dict(layers=96, hidden=12288, seq=2048)
SMALL = dict(layers=8, hidden=2048, seq=1024)
CC_TABLES = 8
MAX_EVALS = 15_905_792 * 256          # op evaluations (ops x scenarios) of the largest listed case
MAX_OPS = 8_000_000                   # ops of a drawn graph: graphs are loaded many times


def _case(name, **kw):
    return dict(DEFAULTS, name=name, **kw)


def listed():
    return [
        # One what-if question about a small job, asked and waited for: launches and latency.
        _case("query-8r-1s", vary="none", check=True),
        # Enumeration of a small job's design space in one batch (the 4096-scenario workload).
        _case("enum-8r-4096s", n=4096),
        # A search loop that reads step times only: no timelines are asked for.
        _case("steps-32r-1000s", **SMALL, tp=4, pp=4, dp=2, mb=8, n=1000, timelines=False),
        # Checked sweep of an odd layout: ragged tiles, two refinements, digests, the
        # allocation-free entry point.
        _case("static-24r-93s", call="static", layers=6, hidden=2048, seq=1024, tp=2, pp=3, dp=4, mb=5, n=93,
              jitter=True, refine=2, digest=True, check=True),
        # GPT-175B on 96 ranks, network sweep (the paper's DDP-study scale).
        _case("gpt175b-96r-64s", **GPT175B, tp=8, pp=4, dp=3, mb=8, n=64, vary="net"),
        # GPT-175B on 1024 ranks, 256 jittered scenarios: the benchmark's default workload.
        _case("gpt175b-1024r-256s", **GPT175B, tp=8, pp=16, dp=8, mb=32, n=256, jitter=True, vary="all"),
        # Extrapolation to large clusters, 32 scenarios: distributed optimizer, TP groups of 4.
        _case("gpt70b-2048r-32s", **GPT70B, tp=4, pp=16, dp=32, mb=16, distopt=True, n=32),
        # The largest job: more ranks than wavefronts, several ranks per walker.
        _case("gpt70b-8192r-32s", **GPT70B, tp=8, pp=16, dp=64, mb=8, n=32),
        # One data-parallel replica standing for the whole job, many scenarios.
        _case("replica-128r-2000s", **GPT175B, tp=8, pp=16, dp=8, mb=8, replica=True, n=2000),
        # The validator iterated to its fixed point, prorated overlaps.
        _case("stable-128r-100s", **GPT70B, tp=4, pp=8, dp=4, mb=8, n=100, jitter=True, refine=16, stable=True,
              prorate=True),
        # Slowdowns predicted by a 64-tree ensemble.
        _case("forest-64r-200s", **GPT70B, tp=8, pp=4, dp=2, mb=8, n=200, jitter=True, forest=True),
        # Collective costs alone, both cost models and profiled tables.
        _case("cc-96r-4000s", call="cc_cost", **GPT175B, tp=8, pp=4, dp=3, mb=8, n=4000, cc="mixed"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the listed ones' ranges: 1 to 1024 ranks (TP 1-8, PP 1-16, DP 1-32), 1 to 32
    microbatches, 1 to 4096 scenarios, every option."""
    while True:
        tp, pp = rng.choice([1, 2, 4, 8]), rng.choice([1, 2, 3, 4, 6, 8, 12, 16])
        c = dict(DEFAULTS, tp=tp, pp=pp, dp=_log(rng, 1, 32), mb=_log(rng, 1, 32), layers=pp * rng.randint(1, 7),
                 hidden=1024 * rng.randint(1, 12), seq=512 * rng.randint(1, 4), distopt=rng.random() < 0.3,
                 n=_log(rng, 1, 4096), jitter=rng.random() < 0.5, vary=rng.choice(["none", "net", "all"]))
        kind = rng.choice(["plain", "plain", "plain", "steps", "digest", "static", "stable", "prorate", "forest",
                           "replica", "cc_cost"])
        c["refine"] = rng.choice([0, 1, 1, 1, 2]) if kind in ("plain", "digest", "static") else 1
        c["cc"] = rng.choice(["echo", "echo", "tables", "mixed"])
        c["check"] = rng.random() < 0.3
        if kind == "steps":
            c["timelines"] = False
        elif kind == "digest":
            c["digest"] = True
        elif kind == "stable":
            c.update(stable=True, refine=rng.randint(2, 16), prorate=rng.random() < 0.5, mb=min(c["mb"], 8))
        elif kind == "prorate":
            c["prorate"] = True
        elif kind == "forest":
            c["forest"] = True
        elif kind == "replica":
            c["replica"] = True
        elif kind in ("static", "cc_cost"):
            c["call"] = kind
        if kind == "cc_cost":
            c["vary"] = rng.choice(["net", "all"])
        ops, colls, _ = _sizes(c)
        whole = _sizes(dict(c, replica=False))[0]
        if whole > MAX_OPS or c["tp"] * c["pp"] * c["dp"] > 1024:
            continue
        if kind == "cc_cost":
            if colls * c["n"] <= 64_000_000:
                return c
        elif kind == "static":
            # the fixed workspace holds one byte per walk item and scenario of whole tiles,
            # and the member slots of collectives that span workgroups
            if 1.5 * ops * (c["n"] + 64) <= 16_000_000:
                return c
        elif ops * c["n"] * (4 if c["stable"] else 1) <= MAX_EVALS:
            return c


def _sizes(case):
    """(ops, collectives, comm ops) of the case's graph, counted from its recipe."""
    T, P, D, m = case["tp"], case["pp"], case["dp"], case["mb"]
    ls, h, seq = case["layers"] // P, case["hidden"], case["seq"]
    ops = colls = comms = 0
    for p in range(P):
        first, last = p == 0, p == P - 1
        ar = 4 * ls + (1 if first else 0) + (3 if last else 0) if T > 1 else 0
        compute = 75 * ls + (3 if first else 0) + (9 if last else 0)
        p2p = 2 * (0 if first else 1) + 2 * (0 if last else 1)
        size = ls * (2 * ((12 * h * h + 13 * h) // T)) + (2 * 2 * h if last else 0) + \
            (2 * (51200 * h // T + seq * h) if first else 0)
        buckets = -(-size // (25 << 20))
        dp = buckets * (2 if case["distopt"] else 1) if D > 1 else 0
        comm = m * (ar + p2p) + dp
        ops += m * (compute + int(first) + int(last)) + buckets + comm
        comms += comm
        colls += m * ar / T + m * p2p / 2 + dp / (1 if case["replica"] else D)
    ranks = T * (1 if case["replica"] else D)
    return ops * ranks, int(round(colls * ranks)), comms * ranks


def _graph(case, seed):
    g = gpt1f1b.gpt_graph(n_layers=case["layers"], hidden=case["hidden"], seq=case["seq"], tp=case["tp"], pp=case["pp"],
                          dp=case["dp"], microbatches=case["mb"], seed=seed, distopt=case["distopt"],
                          replica_invariant=case["replica"])
    return gpt1f1b.dp_replica(g, case["tp"], case["dp"])[0] if case["replica"] else g


def _scenarios(case, seed):
    rng = np.random.default_rng(seed + 1000)
    knobs = {}
    if case["vary"] != "none":
        knobs.update(bw_inter=configs.BW_RANGE, alpha=configs.ALPHA_RANGE)
    if case["vary"] == "all":
        knobs.update(bw_intra=configs.BW_RANGE, ar_algo_random=True, slowdown=configs.SLOWDOWN_RANGE)
    if case["jitter"]:
        knobs.update(jitter=(configs.JITTER_AMP_Q16, seed + 1))
    sc = scenarios.draw(case["n"], rng, **knobs)
    if case["cc"] != "echo":
        sc["cc_table"] = (np.arange(case["n"]) % CC_TABLES + 1).astype(np.int32)
    if case["cc"] == "mixed":
        sc["cc_model"] = (np.arange(case["n"]) % 3 == 0).astype(np.uint8)
        sc["cc_table"][np.arange(case["n"]) % 3 == 1] = 0
    return sc


def _tables(seed):
    return scenarios.draw_cc_tables(CC_TABLES, np.random.default_rng(seed + 2000))


def prepare(case, seed):
    G = E.Graph(_graph(case, seed), 0)
    if case["cc"] != "echo":
        G.set_cc_tables(_tables(seed))
    if case["forest"]:
        G.set_forest(slowdown_forest.synthetic_forest(seed))
    d, n = E.scenarios_to_device(_scenarios(case, seed), "cuda:0")
    out = None
    if case["call"] != "cc_cost" and n > 1:
        # a program that composes many batches keeps its output arrays
        out = {"step": torch.empty(n, dtype=torch.int64, device="cuda:0")}
        if case["timelines"]:
            out["start"] = torch.empty((G.n_ops, n), dtype=torch.int64, device="cuda:0")
            out["finish"] = torch.empty((G.n_ops, n), dtype=torch.int64, device="cuda:0")
        if case["digest"]:
            out["digest"] = torch.empty(n, dtype=torch.int64, device="cuda:0")
    elif case["call"] == "static":
        out = {k: torch.empty((G.n_ops, n) if k in ("start", "finish") else n, dtype=torch.int64, device="cuda:0")
               for k in ("step", "start", "finish", "digest")[:4 if case["digest"] else 3]}
    return {"case": case, "graph": G, "scen": d, "n": n, "out": out}


def run(state):
    c, G = state["case"], state["graph"]
    if c["call"] == "cc_cost":
        return G.cc_cost(state["scen"], state["n"], check=c["check"])
    if c["call"] == "static":
        return G.compose_static(state["scen"], state["n"], c["refine"], state["out"], digest=c["digest"],
                                check=c["check"])
    return G.compose(state["scen"], state["n"], c["refine"], timelines=c["timelines"], digest=c["digest"],
                     out=state["out"], check=c["check"], until_stable=c["stable"], prorate=c["prorate"],
                     forest=c["forest"], refinements=c["stable"])


def work(case):
    """Bytes: outputs written once, the graph (duration, kind, class and predecessor of every op)
    and the scenarios read once.  Operations (64-bit integer): per composed pass a max and an add
    per op and scenario, the jitter draw (two multiplies, three xor-shifts, scaling) once, and
    the divisions of a collective's cost counted as ten each."""
    ops, colls, _ = _sizes(case)
    n = case["n"]
    if case["call"] == "cc_cost":
        return {"bytes": 8 * colls * n + 40 * colls + 192 * n, "flops": 40 * colls * n}
    passes = 1 + (1 if case["stable"] else case["refine"])
    out = (16 * ops if case["timelines"] else 0) + 8 + (8 if case["digest"] else 0)
    return {"bytes": out * n + 16 * ops + 192 * n,
            "flops": ops * n * (2 * passes + (13 if case["jitter"] else 0) + (15 if case["digest"] else 0))}


def tolerance(case):
    return "exact"      # integer nanoseconds throughout


# ------------------------------------------------------------------ plain numpy evaluation
def _costs(g, sc, tables):
    """Cost of every collective in every scenario, [n_colls, n] (int64: no value here nears 2^62)."""
    comm = g["op_kind"] == gpt1f1b.KIND_COMM
    coll, node = g["op_coll"][comm], g["op_rank"][comm] // g["gpus_per_node"]
    nc, n = len(g["coll_type"]), len(sc["alpha_ns"])
    if "coll_N" in g:
        N, M, K = (g[k].astype(np.int64) for k in ("coll_N", "coll_M", "coll_K"))
    else:
        N, M, K = np.bincount(coll, minlength=nc), np.zeros(nc, np.int64), np.zeros(nc, np.int64)
        pair, count = np.unique(np.stack([coll, node], 1), axis=0, return_counts=True)
        np.add.at(M, pair[:, 0], 1)
        np.maximum.at(K, pair[:, 0], count)
    keys, which = np.unique(np.stack([g["coll_type"], g["coll_bytes"], N, M, K], 1).astype(np.int64), axis=0,
                            return_inverse=True)
    div = lambda a, b: -(-a // b)
    tree = sc["ar_algo"] == 1
    intra, inter, red = sc["bw_intra_MBps"], sc["bw_inter_MBps"], sc["reduce_MBps"]
    cost = np.empty((len(keys), n), np.int64)
    for i, (t, S, N_, M_, K_) in enumerate(keys.tolist()):
        # Echo's chunked model: the scenario's bandwidths, or a row of its parameter table
        band = next((j for j, b in enumerate(scenarios.TABLE6_MAX_BYTES) if S <= b), 6)
        if S > scenarios.TABLE6_MAX_BYTES[5]:
            band = 6
        chunk = np.full(n, scenarios.TABLE6_CHUNK[band])
        alpha, r = sc["alpha_ns"].copy(), red.copy()
        beta, gamma = div(chunk * 1000, intra), div(chunk * 1000, inter)
        for s in np.flatnonzero(sc["cc_table"] > 0):
            tb = tables[sc["cc_table"][s] - 1]
            j = next((j for j in range(6) if S <= tb[0, j]), 6)
            chunk[s], alpha[s], beta[s], gamma[s], r[s] = tb[1:, j]
        hop = gamma if M_ > 1 else beta
        ring, chunks, rt = div(S, N_ * chunk), div(S, chunk), div(S * 1000, r)
        if t == gpt1f1b.COLL_AG:
            c = alpha + hop * ring * (N_ - 1)
        elif t == gpt1f1b.COLL_RS:
            c = alpha + ring * (N_ - 1) * (beta + hop) + rt
        elif t == gpt1f1b.COLL_AR:
            c = np.where(tree, alpha + hop * np.maximum(chunks - 1, 0) + 2 * beta * (K_ - 1) +
                         2 * hop * (M_ - 1).bit_length() + rt, alpha + ring * (N_ - 1) * (beta + 2 * hop) + rt)
        else:
            c = alpha + chunks * hop
        # the alpha-beta baseline
        B, part, L = (inter if M_ > 1 else intra), -(-S // N_), (N_ - 1).bit_length()
        a, tb_, tr = sc["alpha_ns"], div(part * 1000, B), div(part * 1000, red)
        whole, wr = div(S * 1000, B), div(S * 1000, red)
        ab = ((N_ - 1) * (a + tb_) if t == gpt1f1b.COLL_AG else (N_ - 1) * (a + tb_ + tr) if t == gpt1f1b.COLL_RS else
              np.where(tree, L * (2 * a + 2 * whole + wr), (N_ - 1) * (2 * a + 2 * tb_ + tr))
              if t == gpt1f1b.COLL_AR else a + whole)
        cost[i] = np.where(sc["cc_model"] == 1, ab, c)
    return cost[which.reshape(-1)]


def _mix(z):
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def _sweep(g, dur, cost):
    """Timelines [n_ops, n]: every op after its stream's previous op and its dependencies; a comm op
    ends when its collective's last member has launched plus the cost."""
    n_ops = len(g["op_rank"])
    off, preds = g["pred_off"], g["pred_idx"]
    start, finish = np.zeros_like(dur), np.zeros_like(dur)
    members = np.bincount(g["op_coll"][g["op_coll"] >= 0], minlength=len(g["coll_type"]))
    prev, tail = np.full(n_ops, -1), {}
    waits, after = np.zeros(n_ops, np.int64), [[] for _ in range(n_ops)]
    for v in range(n_ops):
        k = (int(g["op_rank"][v]), int(g["op_stream"][v]))
        prev[v] = tail.get(k, -1)
        tail[k] = v
        for u in {int(prev[v]), *preds[off[v]:off[v + 1]].tolist()} - {-1}:
            after[u].append(v)
            waits[v] += 1
    ready, joined = [v for v in range(n_ops) if waits[v] == 0], {}
    while ready:
        v = ready.pop()
        for u in {int(prev[v]), *preds[off[v]:off[v + 1]].tolist()} - {-1}:
            np.maximum(start[v], finish[u], out=start[v])
        done, c = [v], int(g["op_coll"][v])
        if c < 0:
            finish[v] = start[v] + dur[v]
        else:
            joined.setdefault(c, []).append(v)
            done = joined[c] if len(joined[c]) == members[c] else []
            for u in done:
                finish[u] = np.max(start[joined[c]], axis=0) + cost[c]
        for u in done:
            for w in after[u]:
                waits[w] -= 1
                if waits[w] == 0:
                    ready.append(w)
    return start, finish


def exact(case, seed):
    """The same outputs from plain numpy, for the collective costs and for small composes with
    whole-op slowdown tables; None elsewhere (a full sweep in Python would take minutes)."""
    ops, colls, _ = _sizes(case)
    if case["stable"] or case["prorate"] or case["forest"] or (case["call"] != "cc_cost" and ops * (1 + case["n"] / 64) > 3e5):
        return None
    g, sc = _graph(case, seed), _scenarios(case, seed)
    cost = _costs(g, sc, _tables(seed))
    if case["call"] == "cc_cost":
        return cost
    n, u64 = case["n"], np.uint64
    v = np.arange(ops, dtype=np.uint64)
    base = np.repeat(g["op_dur"][:, None], n, 1)
    if case["jitter"]:
        amp = sc["jitter_amp_q16"].astype(np.int64)
        k = (sc["jitter_stream"].astype(u64) << u64(36)) + v[:, None] + u64(1)
        high = (_mix(sc["jitter_seed"] + k * u64(0x9E3779B97F4A7C15)) >> u64(32)).astype(np.int64)
        base = (base * (65536 - amp + ((high * (2 * amp + 1)) >> 32)) + 32768) >> 16
    rank, kind = g["op_rank"], g["op_kind"]
    start, finish = _sweep(g, base, cost)
    for _ in range(case["refine"]):
        factor = np.full((ops, n), 65536, np.int64)
        for r in range(g["n_ranks"]):
            comp = np.flatnonzero((rank == r) & (kind == gpt1f1b.KIND_COMPUTE))
            for c in np.flatnonzero((rank == r) & (kind == gpt1f1b.KIND_COMM)):
                hit = np.maximum(start[comp], start[c]) < np.minimum(finish[comp], finish[c])
                f = sc["slowdown_q16"][:, g["op_class"][comp], g["coll_type"][g["op_coll"][c]]].T
                factor[comp] = np.maximum(factor[comp], np.where(hit, f, 65536))
        start, finish = _sweep(g, (base * factor + 32768) >> 16, cost)
    out = {"step": finish.max(axis=0)}
    if case["timelines"]:
        out.update(start=start, finish=finish)
    if case["digest"]:
        out["digest"] = _mix(_mix(v[:, None] ^ start.astype(u64)) ^ finish.astype(u64)).sum(axis=0, dtype=u64).view(np.int64)
    return out
