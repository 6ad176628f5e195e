"""Work that programs built on this runtime have it do, as cases to be timed.

Every case goes through the public binding: a :class:`Runtime` that the
program keeps, jobs submitted to it, one ``run()`` (or one serving session),
results read back.  The kinds:

  batch   fib, N-Queens, UTS and a small k-clique job in one launch
  mix     the job mix of the batching and serving workloads: 60 % k-clique
          jobs (k 4..8) on induced subgraphs of one large power-law graph, 40 %
          UTS jobs (mean 2..4, depth 8..14); batched in one launch or served
          through the admission ring
  kclique k-cliques of one power-law graph: one task per call, or the split
          search with bitset candidate subgraphs (orientation or pivoting)
  fmm     potentials of charged points: work inside the traversal tasks
          (block mode), list-building tasks, or the worklist traversal
  sort    Cilksort of 32-bit keys, one queue or the three DAQ queues
"""
import functools
import math

import torch

from paper_2604_05982_amd import gtap

DEV = "cuda"


def listed():
    return [
        # a handful of tiny jobs: what one call costs (launch, reset, copies, the tree's critical path)
        {"name": "batch_tiny", "kind": "batch", "fib": 12, "queens": 6, "uts_roots": 2, "uts_depth": 5,
         "graph": 2000, "k": 4},
        # the microbenchmarks of the scheduler: many fine tasks, three kinds in one launch
        {"name": "batch_micro", "kind": "batch", "fib": 30, "queens": 12, "uts_roots": 8, "uts_depth": 12,
         "graph": 0, "k": 0},
        # many users' jobs in one persistent launch (the tuned workgroup shape of the job mix)
        {"name": "mix_batched", "kind": "mix", "jobs": 500, "served": False, "waves_per_group": 8},
        # a burst of jobs into a running kernel, through the admission ring (the default workgroup shape)
        {"name": "mix_served", "kind": "mix", "jobs": 200, "served": True, "waves_per_group": 4},
        # k-cliques, one task per call, four divergence-aware queues
        {"name": "kclique7_tasks", "kind": "kclique", "n": 300000, "degree": 40, "k": 7, "search": "tasks",
         "queues": 4},
        # the large k-clique count: split search on the million-vertex graph
        {"name": "kclique7_split", "kind": "kclique", "n": 1000000, "degree": 40, "k": 7, "search": "orient",
         "queues": 1},
        # an ordinary graph, pivoting
        {"name": "kclique6_pivot", "kind": "kclique", "n": 100003, "degree": 30, "k": 6, "search": "pivot",
         "queues": 1},
        # a million clustered points, M2L and P2P inside the traversal tasks
        {"name": "fmm_block_1m", "kind": "fmm", "n": 1000000, "points": "plummer", "leaf": 64, "theta": 2,
         "traversal": "tasks"},
        # an ordinary, ragged point set through the list pipeline
        {"name": "fmm_lists_100k", "kind": "fmm", "n": 100003, "points": "plummer", "leaf": 64, "theta": 2,
         "traversal": "lists"},
        # a large uniform point set through the list pipeline
        {"name": "fmm_lists_4m", "kind": "fmm", "n": 4000000, "points": "uniform", "leaf": 64, "theta": 2,
         "traversal": "lists"},
        # a small sort, one queue
        {"name": "sort_100k", "kind": "sort", "n": 100003, "queues": 1, "bits": 32},
        # a large sort with the recursive / serial sort / serial merge queues
        {"name": "sort_30m", "kind": "sort", "n": 30000000, "queues": 3, "bits": 32},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["batch", "mix", "kclique", "fmm", "sort"])
    if kind == "batch":
        return {"kind": kind, "fib": rng.randint(10, 30), "queens": rng.randint(5, 12),
                "uts_roots": rng.randint(1, 8), "uts_depth": rng.randint(5, 12),
                "graph": _log_int(rng, 500, 20000), "k": rng.randint(3, 6)}
    if kind == "mix":
        return {"kind": kind, "jobs": _log_int(rng, 20, 400), "served": rng.random() < 0.4,
                "waves_per_group": rng.choice([4, 8])}
    if kind == "kclique":
        search = rng.choice(["tasks", "orient", "pivot"])
        return {"kind": kind, "n": _log_int(rng, 2000, 200000 if search == "tasks" else 500000),
                "degree": rng.randint(12, 40), "k": rng.randint(4, 8), "search": search,
                "queues": rng.choice([1, 4])}
    if kind == "fmm":
        traversal = rng.choice(["tasks", "lists", "worklist"])
        return {"kind": kind, "n": _log_int(rng, 2000, 300000 if traversal == "tasks" else 1500000),
                "points": rng.choice(["plummer", "uniform"]), "leaf": rng.choice([32, 48, 64]),
                "theta": rng.choice([2, 3]), "traversal": traversal}
    return {"kind": kind, "n": _log_int(rng, 200, 20000000), "queues": rng.choice([1, 3]),
            "bits": rng.choice([12, 32])}


# ---- inputs ---------------------------------------------------------------------
def _generator(seed, salt=0):
    return torch.Generator(device=DEV).manual_seed((int(seed) * 1000003 + salt) & (2**62 - 1))


def _power_law_edges(n, degree, gamma, cap_frac, gen):
    """Chung-Lu graph oriented by (degree, id): sorted edge arrays u < v of the
    relabelled vertices, int64."""
    b = torch.arange(1, n + 1, dtype=torch.float64, device=DEV).pow(-1.0 / (gamma - 1.0))
    cap = cap_frac * math.sqrt(n * degree)
    lo, hi = 0.0, n * float(degree)
    for _ in range(60):  # the scale at which the capped weights have the mean degree
        c = 0.5 * (lo + hi)
        if float(torch.clamp(c * b, max=cap).mean()) < degree:
            lo = c
        else:
            hi = c
    cdf = torch.cumsum(torch.clamp(hi * b, max=cap), 0)
    m = n * degree // 2
    ends = torch.rand(2, m, dtype=torch.float64, device=DEV, generator=gen) * cdf[-1]
    ends = torch.searchsorted(cdf, ends.reshape(-1)).clamp_(max=n - 1).reshape(2, m)
    a, z = torch.minimum(ends[0], ends[1]), torch.maximum(ends[0], ends[1])
    keys = torch.unique((a * n + z)[a != z])
    a, z = keys // n, keys % n
    deg = torch.bincount(a, minlength=n) + torch.bincount(z, minlength=n)
    pos = torch.empty(n, dtype=torch.int64, device=DEV)
    pos[torch.argsort(deg, stable=True)] = torch.arange(n, device=DEV)
    a, z = pos[a], pos[z]
    keys = torch.sort(torch.minimum(a, z) * n + torch.maximum(a, z)).values
    return keys // n, keys % n


def _csr(n, u, v):
    """int32 out-lists of sorted edges, and the largest out-degree."""
    deg = torch.bincount(u, minlength=n)
    row_ptr = torch.zeros(n + 1, dtype=torch.int32, device=DEV)
    row_ptr[1:] = torch.cumsum(deg, 0)
    col = v.to(torch.int32)
    if col.numel() == 0:
        col = torch.zeros(1, dtype=torch.int32, device=DEV)
    return row_ptr, col, int(deg.max())


@functools.lru_cache(maxsize=1)
def _parent_graph():
    """The graph that the job mix's k-clique jobs take their subgraphs from."""
    return (1000000,) + _power_law_edges(1000000, 40, 2.1, 0.6, _generator(2))


def _subgraph(n, u, v, s, gen):
    """The subgraph induced on s random vertices, renumbered in order."""
    new = torch.full((n,), -1, dtype=torch.int64, device=DEV)
    picked = torch.sort(torch.randperm(n, device=DEV, generator=gen)[:s]).values
    new[picked] = torch.arange(s, device=DEV)
    a, z = new[u], new[v]
    keep = (a >= 0) & (z >= 0)
    return _csr(s, a[keep], z[keep])


def _points(n, law, gen):
    def rand():
        return torch.rand(n, dtype=torch.float64, device=DEV, generator=gen)

    if law == "uniform":
        x, y, z = (200.0 * rand() - 100.0 for _ in range(3))
    else:  # Plummer sphere of scale 1, radius at most 100
        r = 1.0 / torch.sqrt((rand() * (1 - 1e-9) + 1e-9).mul_(0.9998).pow(-2.0 / 3.0) - 1.0)
        c = 2.0 * rand() - 1.0
        t = 2.0 * math.pi * rand()
        s = torch.sqrt(1.0 - c * c)
        x, y, z = (a.clamp(-100.0, 100.0) for a in (r * s * torch.cos(t), r * s * torch.sin(t), r * c))
    return [a.contiguous() for a in (x, y, z, 2.0 * rand() - 1.0)]


def _keys(case, seed):
    return torch.randint(-2**31 if case["bits"] == 32 else 0, 2**31 if case["bits"] == 32 else 2**case["bits"],
                         (case["n"],), dtype=torch.int64, device=DEV, generator=_generator(seed)).to(torch.int32)


# ---- prepare / run -----------------------------------------------------------------
def prepare(case, seed):
    gen = _generator(seed)
    state = {"case": case}
    kind = case["kind"]
    if kind == "batch":
        big = 0
        if case["graph"]:
            n = case["graph"]
            row_ptr, col, big = _csr(n, *_power_law_edges(n, 16, 2.5, 1.0, gen))
            state["graph"] = (row_ptr, col, big)
        state["uts"] = [int(s) for s in torch.randint(1, 2**62, (case["uts_roots"],), device=DEV, generator=gen)]
        state["rt"] = gtap.Runtime(waves_per_group=4, small_frames=1 << 24, big_frames=1 << 18,
                                   big_frame_ints=max(64, big), timeout_ms=60000)
    elif kind == "mix":
        jobs, keep, big = [], [], 64
        parent = _parent_graph()
        shape = torch.rand(case["jobs"], 4, device=DEV, generator=gen, dtype=torch.float64).tolist()
        ids = torch.randint(1, 2**62, (case["jobs"],), device=DEV, generator=gen).tolist()
        for (a, b, c, d), ident in zip(shape, ids):
            if a < 0.6:
                graph = _subgraph(*parent, int(round(1000 * 200.0 ** b)), gen)
                big = max(big, graph[2])
                jobs.append(("kclique", graph, 4 + int(5 * c)))
            else:
                jobs.append(("uts", ident, gtap.uts_threshold(2.0 + 2.0 * b), 8 + int(7 * c)))
        rt = gtap.Runtime(waves_per_group=case["waves_per_group"],
                          num_waves=0 if case["waves_per_group"] == 8 else 1024, max_jobs=4096,
                          small_frames=1 << 26, big_frames=1 << 21, big_frame_ints=big, deque_capacity=1 << 17,
                          timeout_ms=60000)
        if case["served"]:
            state["trace"] = rt.trace([
                (0.0, rt.kclique_args(j[1][0], j[1][1], j[2], max_outdeg=j[1][2]) if j[0] == "kclique"
                 else rt.uts_args(*j[1:])) for j in jobs])
        state["rt"], state["jobs"] = rt, jobs
    elif kind == "kclique":
        n = case["n"]
        row_ptr, col, big = _csr(n, *_power_law_edges(n, case["degree"], 2.1, 0.6, gen))
        state["graph"] = (row_ptr, col, big)
        opts = {}
        if case["queues"] > 1:
            opts = dict(num_queues=case["queues"], daq_policy=gtap.GTAP_DAQ_KCLIQUE, daq_bounds=[8, 32, 128])
        ints = max(64, big) if case["search"] == "tasks" else gtap.kclique_split_buffer_ints(big)
        state["rt"] = gtap.Runtime(num_waves=1024, waves_per_group=4, small_frames=1 << 25, big_frames=1 << 23,
                                   big_frame_ints=ints, deque_capacity=1 << (18 if case["queues"] > 1 else 17),
                                   timeout_ms=60000, **opts)
    elif kind == "fmm":
        state["points"] = _points(case["n"], case["points"], gen)
        state["phi"] = torch.zeros(case["n"], dtype=torch.float64, device=DEV)
        if case["traversal"] == "tasks":
            state["rt"] = gtap.Runtime(mode=gtap.GTAP_MODE_BLOCK, waves_per_group=2, small_frames=1 << 24,
                                       big_frames=0, timeout_ms=60000)
        else:
            state["rt"] = gtap.Runtime(mode=gtap.GTAP_MODE_THREAD, waves_per_group=4, small_frames=1 << 24,
                                       big_frames=1 << 10, timeout_ms=60000)
    else:
        opts = {}
        if case["queues"] > 1:
            opts = dict(num_queues=case["queues"], daq_policy=gtap.GTAP_DAQ_CILKSORT)
        state["source"] = _keys(case, seed)
        state["keys"] = torch.empty_like(state["source"])
        state["tmp"] = torch.empty_like(state["source"])
        state["rt"] = gtap.Runtime(waves_per_group=4, small_frames=1 << 24, big_frames=1 << 10,
                                   deque_capacity=1 << 17, timeout_ms=60000, **opts)
    return state


_TRAVERSALS = {"tasks": gtap.GTAP_FMM_TASKS, "lists": gtap.GTAP_FMM_LISTS, "worklist": gtap.GTAP_FMM_WORKLIST}


def run(state):
    case, rt = state["case"], state["rt"]
    kind = case["kind"]
    if kind == "batch":
        jobs = [rt.submit_fib(case["fib"]), rt.submit_nqueens(case["queens"])]
        jobs += [rt.submit_uts(s, gtap.uts_threshold(4), case["uts_depth"]) for s in state["uts"]]
        if case["graph"]:
            row_ptr, col, big = state["graph"]
            jobs.append(rt.submit_kclique(row_ptr, col, case["k"], max_outdeg=big))
        rt.run()
        return torch.tensor([rt.result(j) for j in jobs])
    if kind == "mix":
        if case["served"]:
            rt.serve_start(max_inflight=1024, headroom_small=1 << 22)
            served = rt.trace_run(state["trace"])
            rt.serve_stop()
            return torch.tensor([r.result for r in served])
        ids = [rt.submit_kclique(j[1][0], j[1][1], j[2], max_outdeg=j[1][2]) if j[0] == "kclique"
               else rt.submit_uts(*j[1:]) for j in state["jobs"]]
        rt.run()
        return torch.tensor([rt.result(j) for j in ids])
    if kind == "kclique":
        row_ptr, col, big = state["graph"]
        if case["search"] == "tasks":
            job = rt.submit_kclique(row_ptr, col, case["k"], max_outdeg=big)
        else:
            job = rt.submit_kclique_split(row_ptr, col, case["k"], threshold=64, max_outdeg=big,
                                          algorithm=gtap.GTAP_KCLIQUE_PIVOT if case["search"] == "pivot"
                                          else gtap.GTAP_KCLIQUE_ORIENT)
        rt.run()
        return rt.result(job)
    if kind == "fmm":
        job = rt.submit_fmm(*state["points"], state["phi"], leaf_max=case["leaf"], theta=(1, case["theta"]),
                            traversal=_TRAVERSALS[case["traversal"]])
        rt.run()
        res = rt.fmm_result(job)
        return {"phi": state["phi"], "cells": res["n_cells"], "m2l": res["m2l_pairs"], "p2p": res["p2p_pairs"],
                "interactions": res["p2p_interactions"]}
    # the sort is in place: the program's keys arrive in the buffer first
    state["keys"].copy_(state["source"])
    job = rt.submit_cilksort(state["keys"], state["tmp"])
    rt.run()
    return {"keys": state["keys"], "count": rt.result(job)}


# ---- what a pass cannot do without ---------------------------------------------------
def _uts_nodes(mean, depth):
    return depth + 1.0 if mean == 1 else (mean ** (depth + 1) - 1.0) / (mean - 1.0)


def work(case):
    """Integer operations are counted as flops.  Job sizes that depend on the
    drawn inputs are expected values."""
    kind = case["kind"]
    if kind == "batch":
        fib = 2.0 * 1.618034 ** (case["fib"] + 1) / math.sqrt(5.0)          # calls
        queens = 0.0065 * math.factorial(case["queens"]) ** 0.97             # search nodes, roughly
        uts = case["uts_roots"] * _uts_nodes(4.0, case["uts_depth"])
        graph = 8.0 * case["graph"]                                          # oriented edges
        # a call: an addition and a test; a node: masks and a test per column;
        # a tree node: about three 64-bit hashes of 20 operations
        return {"bytes": 4.0 * (graph + case["graph"] + 1) + 8.0, "flops": 4 * fib + 12 * queens + 60 * uts + 16 * graph}
    if kind == "mix":
        # means over the law of the jobs (mean 2..4, depth 8..14): 9.4 M nodes a UTS job;
        # a k-clique job has 3.8e4 vertices and 2.4e5 edges
        uts, kcl = 0.4 * case["jobs"], 0.6 * case["jobs"]
        return {"bytes": kcl * 4.0 * (3.8e4 + 2.4e5) + 8.0 * case["jobs"], "flops": uts * 9.4e6 * 60 + kcl * 2.4e5 * 16}
    if kind == "kclique":
        edges = case["n"] * case["degree"] / 2.0
        # the triangles alone: per edge the shorter of two out-lists
        return {"bytes": 4.0 * (case["n"] + 1 + edges) + 8.0, "flops": edges * case["degree"]}
    if kind == "fmm":
        n, scale = float(case["n"]), (case["theta"] / 2.0) ** 3
        near = min(n, (6000.0 if case["points"] == "plummer" else 2500.0) * scale * case["leaf"] / 64.0)
        far = 40.0 * scale * 64.0 / case["leaf"]
        # 20 operations a near interaction, 924 multiply-adds and the 84 derivatives a far pair
        return {"bytes": 8.0 * 5 * n, "flops": n * (20.0 * near + 2448.0 * far)}
    n = float(case["n"])
    return {"bytes": 8.0 * n + 8.0 * n, "flops": n * max(1.0, math.log2(n))}  # the copy in, then read and written once


def exact(case, seed):
    if case["kind"] == "sort":
        keys = torch.sort(_keys(case, seed).to(torch.int64) & 0xFFFFFFFF).values
        keys = torch.where(keys >= 2**31, keys - 2**32, keys).to(torch.int32)
        return {"keys": keys, "count": case["n"]}
    if case["kind"] == "fmm" and case["n"] <= 150000:
        x, y, z, q = _points(case["n"], case["points"], _generator(seed))
        phi = torch.empty_like(x)
        step = max(1, (1 << 27) // case["n"])
        for i in range(0, case["n"], step):
            e = min(case["n"], i + step)
            r2 = (x[i:e, None] - x[None]).square_()
            r2 += (y[i:e, None] - y[None]).square_()
            r2 += (z[i:e, None] - z[None]).square_()
            r2[r2 == 0.0] = math.inf
            phi[i:e] = r2.rsqrt_() @ q
        return {"phi": phi, "cells": None, "m2l": None, "p2p": None, "interactions": None}
    return None
