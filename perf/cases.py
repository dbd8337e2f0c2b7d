"""Performance cases of the simulator: what its users run, from one tiny
collective (launch and per-cycle latency) to batched design sweeps, large
single topologies and GPU-as-NoC programs.

A case names a topology family, a workload and sizes; the link parameters
come from the seed.  ``prepare`` builds the topology, loads the workload and
allocates the output buffers (what a program keeps between runs), ``run``
enqueues one full simulation of every scenario and hands out the four output
arrays.  All outputs are whole numbers (cycles and counts), so they are
compared exactly.
"""
from __future__ import annotations

import math
from dataclasses import replace

import numpy as np

import sim_inputs as si
from sim_inputs import noc
from paper_2606_10440_amd.sim import Simulator

COLLS = {"ring": si.COLL_RING_ALLREDUCE, "direct": si.COLL_DIRECT_ALLREDUCE, "hier": si.COLL_HIER_ALLREDUCE,
         "alltoall": si.COLL_ALLTOALL, "ring_ag": si.COLL_RING_ALLGATHER, "ring_rs": si.COLL_RING_REDUCESCATTER,
         "rhd": si.COLL_RHD_ALLREDUCE, "dbt": si.COLL_DBT_ALLREDUCE}
ARBS = {"lowest": si.ARB_LOWEST_ID, "rr": si.ARB_ROUND_ROBIN}
LINE = si.LINE_BYTES


def listed():
    return [
        # one small collective inside a scale-up domain: a run of a few hundred cycles
        {"name": "mesh4_direct_64k", "kind": "mesh", "p": 4, "coll": "direct", "lines": 512, "b": 1, "lat": 10,
         "cap": 16, "arb": "lowest"},
        # one long collective on one node: hundreds of thousands of dependent cycles, few links
        {"name": "mesh8_ring_16m", "kind": "mesh", "p": 8, "coll": "ring", "lines": 131072, "b": 1, "lat": 50,
         "cap": 64, "arb": "lowest"},
        # the batched design sweep: thousands of bandwidth / latency / depth points of one torus
        {"name": "torus4x4_ring_4m_x4096", "kind": "torus", "X": 4, "Y": 4, "coll": "ring", "lines": 32768,
         "S": 4096, "dep": 0, "credit": False, "arb": "lowest"},
        # the same sweep with per-chunk (put + signal) steps
        {"name": "torus4x4_ring_chunk_x2048", "kind": "torus", "X": 4, "Y": 4, "coll": "ring", "lines": 4096,
         "S": 2048, "dep": 1, "credit": False, "arb": "lowest"},
        # tree all-reduce over the sweep: every link shared by several flows
        {"name": "torus4x4_dbt_1m_x4096", "kind": "torus", "X": 4, "Y": 4, "coll": "dbt", "lines": 8192,
         "S": 4096, "dep": 0, "credit": False, "arb": "lowest"},
        # halving-doubling over a smaller sweep, credits that travel back over the link
        {"name": "torus4x4_rhd_credit_x1024", "kind": "torus", "X": 4, "Y": 4, "coll": "rhd", "lines": 8192,
         "S": 1024, "dep": 0, "credit": True, "arb": "lowest"},
        # a design sweep of a small cluster fabric, all-to-all (expert-parallel traffic): many flows per link
        {"name": "fattree4_sweep_x512", "kind": "fattree", "k": 4, "lines": 128, "cap": 0, "credit": False, "S": 512},
        # scale-up domains behind a leaf/spine fabric: hierarchical all-reduce
        {"name": "hier8x8_4m", "kind": "hier", "G": 8, "M": 8, "leaf": 8, "spine": 4, "lines": 32768},
        # one fat-tree cluster, all-to-all
        {"name": "fattree8_alltoall_8k", "kind": "fattree", "k": 8, "lines": 64, "cap": 32, "credit": False, "S": 1},
        # the same cluster with credit-based flow control
        {"name": "fattree8_credit_8k", "kind": "fattree", "k": 8, "lines": 64, "cap": 32, "credit": True, "S": 1},
        # two GPUs as networks on chip: put-based all-gather by memcpy programs, swept over memory and cable latencies
        {"name": "noc2_allgather_1m_x512", "kind": "noc", "G": 2, "op": "ag_put", "lines": 8192, "S": 512, "unroll": 4,
         "window": 64},
        # eight GPUs as networks on chip, one run: get-based reduce-scatter
        {"name": "noc8_reducescatter_128k", "kind": "noc", "G": 8, "op": "rs_get", "lines": 1024, "S": 1, "unroll": 4,
         "window": 64},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["mesh", "mesh", "torus", "torus", "torus", "torus", "hier", "fattree", "fattree", "noc", "noc",
                       "noc"])
    if kind == "mesh":  # domains of 3 to 12 endpoints, a few lines to tens of thousands per endpoint
        p = rng.randint(3, 12)
        coll = rng.choice(["direct", "ring", "ring_ag", "alltoall", "dbt"] + (["rhd"] if p & (p - 1) == 0 else []))
        c = _log(rng, 8, 6000)
        lines = max(1, c // p) if coll == "alltoall" else 2 * max(1, c // 2) * p
        return {"kind": "mesh", "p": p, "coll": coll, "lines": lines, "b": rng.choice([1, 1, 2, 4]),
                "lat": rng.randint(5, 100), "cap": rng.choice([16, 24, 32, 64]), "arb": rng.choice(["lowest", "rr"])}
    if kind == "torus":  # design sweeps over 3x2 to 6x5 tori
        # (all-pairs exchanges on a torus can deadlock on its cyclic buffers and are left out)
        X, Y = rng.randint(2, 6), rng.randint(2, 5)
        p = X * Y
        coll = rng.choice(["ring", "ring", "ring_rs", "dbt"] + (["rhd"] * 2 if p & (p - 1) == 0 else []))
        S = _log(rng, 16, 4096 if p <= 16 else 512)
        lines = p * (2 if coll == "dbt" else 1) * _log(rng, 16, 1000 if p <= 16 else 300)
        credit = rng.random() < 0.2
        return {"kind": "torus", "X": X, "Y": Y, "coll": coll, "lines": lines, "S": S,
                "dep": 0 if credit else int(rng.random() < 0.25), "credit": credit,
                "arb": rng.choice(["lowest", "lowest", "rr"])}
    if kind == "hier":  # 2 to 8 domains of 2 to 8 endpoints
        G, M = rng.randint(2, 8), rng.randint(2, 8)
        return {"kind": "hier", "G": G, "M": M, "leaf": G, "spine": rng.choice([2, 3, 4]),
                "lines": G * M * _log(rng, 8, 400)}
    if kind == "fattree":  # a sweep of 16 hosts, or one cluster of 16 to 128
        if rng.random() < 0.35:
            return {"kind": "fattree", "k": 4, "lines": _log(rng, 4, 128), "cap": 0, "credit": False,
                    "S": _log(rng, 16, 512)}
        k = rng.choice([4, 6, 8])
        return {"kind": "fattree", "k": k, "lines": _log(rng, 2, 48 if k == 8 else 96), "cap": rng.choice([16, 32, 64]),
                "credit": rng.random() < 0.4, "S": 1}
    G = rng.choice([2, 2, 2, 3, 4])
    op = rng.choice(["ag_put", "ag_get", "rs_get", "rs_put", "alltoall"])
    S = _log(rng, 1, 400) if G == 2 else 1
    slices = _log(rng, 1, 16 if S > 64 else 32)  # lines per workgroup slice
    return {"kind": "noc", "G": G, "op": op, "lines": 32 * slices * (1 if op == "alltoall" else G), "S": S,
            "unroll": rng.choice([1, 2, 4, 8]), "window": rng.choice([16, 64, 256])}


def _workload(c, seed):
    """The case's topology, link parameters (drawn from the seed) and workload."""
    r = np.random.RandomState(seed % (1 << 32))
    if c["kind"] == "mesh":
        w = si.full_mesh(c["p"], b=c["b"], L=c["lat"], cap=c["cap"], coll=COLLS[c["coll"]],
                         nbytes=c["lines"] * LINE, arb=ARBS[c["arb"]])
        w.lat = r.randint(c["lat"], c["lat"] + max(1, c["lat"] // 4) + 1, w.n_links).astype(np.int32)
        return w
    if c["kind"] == "torus":
        w = si.torus2d(c["X"], c["Y"], n_scenarios=c["S"], seed=seed, nbytes=c["lines"] * LINE, coll=COLLS[c["coll"]],
                       arb=ARBS[c["arb"]])
        X, Y = c["X"], c["Y"]
        if c["coll"] == "rhd" and X & (X - 1) == 0 and Y & (Y - 1) == 0:
            w = replace(w, order=si.gray_torus_order(X, Y))
        return replace(w, dep=c["dep"], credit=w.lat.copy() if c["credit"] else None)
    if c["kind"] == "hier":
        w = si.domains_leaf_spine(c["G"], c["M"], c["leaf"], c["spine"], nbytes=c["lines"] * LINE)
        w.lat = (w.lat + r.randint(0, 1 + w.lat // 4)).astype(np.int32)
        return w
    if c["kind"] == "fattree":
        w = si.fat_tree(c["k"], lat_seed=seed, cap=c["cap"], nbytes=c["lines"] * LINE)
        S, m = c["S"], w.n_links
        if S > 1:  # one (bandwidth, latency scale, depth) point per scenario
            lat = r.randint(20, 201, S)[:, None] * w.lat[None, :] // 200
            return replace(w, n_scenarios=S, lat=lat.astype(np.int32).reshape(-1),
                           bw=np.repeat(r.choice([1, 2, 4], S), m).astype(np.int32),
                           cap=np.repeat(r.choice([16, 32, 64], S), m).astype(np.int32))
        return replace(w, credit=w.lat.copy()) if c["credit"] else w
    w, lay = noc.gpu_noc(c["G"])
    kw = {"unroll": c["unroll"], "window": c["window"]}
    ops = {"ag_put": lambda: noc.allgather_ops(lay, c["lines"], **kw),
           "ag_get": lambda: noc.allgather_ops(lay, c["lines"], get=True, **kw),
           "rs_get": lambda: noc.reducescatter_ops(lay, c["lines"], get=True, **kw),
           "rs_put": lambda: noc.reducescatter_ops(lay, c["lines"], get=False, **kw),
           "alltoall": lambda: noc.alltoall_ops(lay, c["lines"], **kw)}[c["op"]]()
    return noc.with_scenarios(noc.memcpy_workload(w, ops), c["S"], seed)


def prepare(case, seed):
    sim = Simulator.from_workload(_workload(case, seed))
    return {"sim": sim, "outs": sim.alloc_outputs()}


def run(state):
    state["sim"].enqueue(state["outs"])
    return state["outs"]


def _sizes(c):
    """(lines, links, scenarios) of a case."""
    n, S = c["lines"], c.get("S", 1)
    if c["kind"] == "noc":
        G, wg = c["G"], 32
        T = {"ag_put": 3 * G * n, "ag_get": 3 * G * n, "alltoall": 3 * G * (G - 1) * n, "rs_get": (2 * G + 1) * n,
             "rs_put": 3 * (G - 1) * n + 3 * G * (G - 1) * wg + (2 * G + 1) * n}[c["op"]]
        return T, 1000 * G, S
    if c["kind"] == "mesh":
        p, m = c["p"], c["p"] * (c["p"] - 1)
    elif c["kind"] == "torus":
        p = c["X"] * c["Y"]
        m = p * sum(0 if d == 1 else 1 if d == 2 else 2 for d in (c["X"], c["Y"]))
    elif c["kind"] == "hier":
        G, M = c["G"], c["M"]
        ring = (2 * G - 2) * G * M * (n // M // G)
        return 2 * (M - 1) * G * n + ring, G * M * (M - 1) + 2 * G * M + 2 * c["leaf"] * c["spine"], 1
    else:
        H = c["k"] ** 3 // 4
        return H * (H - 1) * n, 6 * H, S
    T = {"ring": 2 * (p - 1) * n, "direct": 2 * (p - 1) * n, "ring_ag": (p - 1) * n, "ring_rs": (p - 1) * n,
         "alltoall": p * (p - 1) * n, "rhd": 2 * (p - 1) * n, "dbt": 2 * (p - 1) * n}
    return T[c["coll"]], m, S


def work(case):
    # a completion cycle per line, two counters per link, the makespan; three
    # parameters read per link (the queue work itself has no arithmetic rate)
    T, m, S = _sizes(case)
    return {"bytes": S * (4 * T + 16 * m + 4 + 12 * m), "flops": 0}


def tolerance(case):
    return "exact"


def exact(case, seed):
    """Ring and direct all-reduce on a full mesh, where every flow has a link
    of its own: line k of a link enters it at the latest of its release, the
    line before it, the bandwidth (b per cycle) and the slot of line k - cap;
    it leaves after the latency, in order, b per cycle.  Other cases: None
    (whole numbers, compared exactly)."""
    if case["kind"] != "mesh" or case["coll"] not in ("ring", "direct"):
        return None
    p, b, cap = case["p"], case["b"], case["cap"]
    C = case["lines"] // p
    T, m, _ = _sizes(case)
    if T > 4_000_000:
        return None
    w = _workload(case, seed)
    link = {}
    for u in range(p):
        for q in range(w.row_ptr[u], w.row_ptr[u + 1]):
            link[u, int(w.col_idx[q])] = q
    comp = [0] * T
    adm = [[] for _ in range(m)]
    dep = [[] for _ in range(m)]

    def send(u, v, first, rel):
        q = link[u, v]
        A, D, L = adm[q], dep[q], int(w.lat[q])
        for j in range(C):
            k = len(A)
            a = rel[j]
            if k:
                a = max(a, A[-1])
            if k >= b:
                a = max(a, A[k - b] + 1)
            if k >= cap:
                a = max(a, D[k - cap] + 1)
            d = a + L
            if k:
                d = max(d, D[-1])
            if k >= b:
                d = max(d, D[k - b] + 1)
            A.append(a)
            D.append(d)
            comp[first + j] = d + 1

    none = [0] * C
    if case["coll"] == "ring":
        for s in range(2 * p - 2):
            for i in range(p):
                at = ((s - 1) * p + (i - 1) % p) * C
                send(i, (i + 1) % p, (s * p + i) * C, comp[at:at + C] if s else none)
    else:
        for ph in range(2):
            for k in range(1, p):
                for i in range(p):
                    rel = none
                    if ph:
                        into = [(((i - x) % p - 1) * p + x) * C for x in range(p) if x != i]
                        rel = [max(comp[at + j] for at in into) for j in range(C)]
                    send(i, (i + k) % p, ((ph * (p - 1) + k - 1) * p + i) * C, rel)
    return (np.array([comp], np.float64), np.array([[len(a) for a in adm]], np.float64),
            np.array([[len(set(a)) for a in adm]], np.float64), np.array([max(comp)], np.float64))
