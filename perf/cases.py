"""Workloads of the move evaluator: what a program that searches with it has it do.

A case is one pass through the public entry points of ``paper_2506_17357_amd``:

* ``query``   one best move of a solution held on the device (the call a host-driven search makes per
              iteration; the smallest work there is, so latency and launches count).
* ``search``  one local search of a solution: new routes in, ``steps`` device-resident steps, routes out.
              ``mode`` is the neighbourhood: plain (the five operators), granular (theta nearest
              neighbours), penalised (infeasible solutions allowed), variants (segment relocations and
              cross-exchanges as well) or multi (several independent moves per step).  Problems are CVRP,
              VRPTW and VRPSPDTW (pickups).
* ``batch``   a population improved together: new routes for every member, ``steps`` steps of all of them
              in one batch, every member's routes out.
* ``served``  the serving engine's inner loop: members of very different sizes on the whole-LDS schedule
              of the server, advanced by ticks of four steps.
* ``setup``   a new instance taken up: distances and nodes registered and checked, neighbour lists built,
              a first solution set, its first best moves.

Sizes follow the repository's own instances and request streams: 100 to 2000 customers in populations, 200
to 10^4 customers per served request, 1000 customers for the operator extensions.  Searches stop after
``steps`` steps, fewer than a search from a sweep solution takes to its local optimum, so that every step
does its whole work.
"""
import math

import numpy as np
import torch

from paper_2506_17357_amd import tga
from paper_2506_17357_amd import workload as wl

MASKS = {"plain": tga.OPS_ALL, "granular": tga.OPS_ALL | tga.OP_GRANULAR, "penalised": tga.OPS_ALL,
         "variants": tga.OPS_ALL | tga.OPS_VARIANTS, "multi": tga.OPS_ALL | tga.OP_MULTI}


def listed():
    return [
        # a small delivery round optimised interactively, one best-move call after another: pure latency
        {"name": "query-cvrp-100", "form": "query", "problem": "cvrp", "n": 100},
        # the same call on the 1000-customer clustered instance with windows
        {"name": "query-vrptw-1000", "form": "query", "problem": "vrptw", "n": 1000},
        # a small instance improved on the device: the step's fixed costs
        {"name": "search-vrptw-201", "form": "search", "problem": "vrptw", "n": 201, "mode": "plain", "steps": 50},
        # the 1000-customer instances, one solution at a time, in each neighbourhood
        {"name": "search-cvrp-1000", "form": "search", "problem": "cvrp", "n": 1000, "mode": "plain", "steps": 200},
        {"name": "granular-vrptw-1000", "form": "search", "problem": "vrptw", "n": 1000, "mode": "granular",
         "theta": 100, "steps": 200},
        {"name": "penalised-vrptw-1000", "form": "search", "problem": "vrptw", "n": 1000, "mode": "penalised",
         "steps": 100},
        {"name": "variants-cvrp-997", "form": "search", "problem": "cvrp", "n": 997, "mode": "variants", "steps": 100},
        {"name": "multi-vrptw-1000", "form": "search", "problem": "vrptw", "n": 1000, "mode": "multi", "steps": 16},
        {"name": "pickups-vrpspdtw-603", "form": "search", "problem": "vrpspdtw", "n": 603, "mode": "plain",
         "steps": 100},
        # a population of a memetic search: CVRP and VRPTW mixed, uneven sizes
        {"name": "batch-256", "form": "batch", "count": 256, "lo": 100, "hi": 2000, "steps": 200},
        # the serving engine with requests of every size, the largest included
        {"name": "served-16", "form": "served", "count": 16, "lo": 200, "hi": 10000, "ticks": 8},
        # a new mid-size instance
        {"name": "setup-vrptw-2500", "form": "setup", "problem": "vrptw", "n": 2500, "theta": 50},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    form = rng.choice(["query", "search", "search", "search", "search", "batch", "served", "setup"])
    if form == "query":
        return {"form": form, "problem": rng.choice(["cvrp", "vrptw"]), "n": _log_int(rng, 50, 5000)}
    if form == "search":
        mode = rng.choice(["plain", "granular", "penalised", "variants", "multi"])
        problem = rng.choice(["cvrp", "vrptw"] if mode == "granular" else ["cvrp", "vrptw", "vrpspdtw"])
        n = _log_int(rng, 60, 2500 if mode in ("plain", "granular") else 1500)
        case = {"form": form, "problem": problem, "n": n, "mode": mode,
                "steps": max(2, n // 60) if mode == "multi" else rng.randint(max(2, n // 20), max(3, n // 5))}
        if mode == "granular":
            case["theta"] = rng.randint(10, min(100, n // 2))
        return case
    if form == "batch":
        lo = _log_int(rng, 60, 400)
        return {"form": form, "count": _log_int(rng, 8, 128), "lo": lo, "hi": rng.randint(2 * lo, 1600),
                "steps": rng.randint(10, max(11, lo // 5))}
    if form == "served":
        return {"form": form, "count": rng.randint(1, 12), "lo": _log_int(rng, 100, 600), "hi": _log_int(rng, 700, 8000),
                "ticks": rng.randint(2, 5)}
    n = _log_int(rng, 80, 2500)
    return {"form": form, "problem": rng.choice(["cvrp", "vrptw"]), "n": n, "theta": rng.randint(5, min(100, n // 2))}


# ------------------------------------------------------------------- inputs --

def _instance(problem, n, seed):
    if problem == "cvrp":  # the small instance's demands, or the 1000-customer one's
        inst = wl.make_cvrp(n, seed, demand_max=10, capacity=50) if n <= 150 else wl.make_cvrp(n, seed)
    elif problem == "vrptw":
        inst = wl.make_vrptw(n, seed)
    else:
        inst = wl.make_vrpspdtw(n, seed)
    return inst, wl.sweep(inst)


def _sizes(case):
    """Sizes spread evenly over the logarithm of [lo, hi], the largest first."""
    c, lo, hi = case["count"], case["lo"], case["hi"]
    if c == 1:
        return [hi]
    return [int(round(hi * (lo / hi) ** (i / (c - 1)))) for i in range(c)]


class _State:
    pass


def _members(case, seed):
    out = []
    for i, n in enumerate(_sizes(case)):
        inst, sol = _instance("cvrp" if i % 2 == 0 else "vrptw", n, 100003 * seed + i)
        out.append((tga.Instance.from_workload(inst), sol))
    return out


def prepare(case, seed):
    st = _State()
    st.case = case
    form = case["form"]
    if form in ("batch", "served"):
        members = _members(case, seed)
        st.routes = [s for _, s in members]
        st.sols = [tga.Solution(I, s.offsets, s.customers) for I, s in members]
        if form == "batch":
            # the schedule the autotuner settles on for such mixes
            st.batch = tga.Batch(st.sols)
            st.batch.set_config(79, 0)
        else:
            # the server's schedule: one inter-route workgroup per compute unit
            st.batch = tga.SlotBatch(len(st.sols) + 2, sum(s.Q for s in st.sols) + 64, sum(s.R for s in st.sols) + 8)
            st.batch.set_config(tga.device_limits()[1] // 1024, 0)
            st.batch.set_members(st.sols + [None, None])
        return st
    inst, sol = _instance(case["problem"], case["n"], seed)
    st.routes = sol
    if form == "setup":
        st.inst = inst
        st.dist = torch.as_tensor(inst.dist).cuda()
        st.node4 = torch.as_tensor(inst.node4).cuda()
        return st
    st.inst = tga.Instance.from_workload(inst)
    mode = case.get("mode", "plain")
    if mode == "granular":
        st.inst.set_granular(case["theta"])
    st.sol = tga.Solution(st.inst, sol.offsets, sol.customers)
    if mode == "penalised":
        st.sol.set_penalty(10, 0 if case["problem"] == "cvrp" else 10)
    elif mode == "variants":
        st.sol.set_general(True)
    elif mode == "multi":
        st.sol.set_multi(True)
    return st


# --------------------------------------------------------------------- pass --

def _move(m):
    return [0] * 6 if m is None else [m.op, m.k, m.a, m.b, m.delta, m.id]


def _tour(solutions):
    """Routes read back from the device: the customers in order, and the route each of them is on."""
    got = [s.get() for s in solutions]
    return {"customers": np.concatenate([c for _, c, _ in got]),
            "route": np.concatenate([np.repeat(np.arange(len(o) - 1), np.diff(o)) for o, _, _ in got]),
            "cost": np.array([c for _, _, c in got])}


def run(st):
    case = st.case
    form = case["form"]
    if form == "query":
        return _move(st.sol.eval())
    if form == "search":
        st.sol.reload(st.routes.offsets, st.routes.customers)
        steps, moves, _ = st.sol.ls_run(case["steps"], MASKS[case["mode"]])
        return dict(_tour([st.sol]), steps=steps, moves=moves)
    if form == "batch":
        for s, r in zip(st.sols, st.routes):
            s.reload(r.offsets, r.customers)
        steps, moves, _ = st.batch.ls_run(case["steps"])
        return dict(_tour(st.sols), steps=steps, moves=moves)
    if form == "served":
        for s, r in zip(st.sols, st.routes):
            s.reload(r.offsets, r.customers)
            s.begin(500)
        for _ in range(case["ticks"]):
            st.batch.tick(4)
        return _tour(st.sols)
    inst = tga.Instance(st.inst.n, st.dist, st.node4, st.inst.capacity, st.inst.has_tw)
    inst.set_granular(case["theta"])
    sol = tga.Solution(inst, st.routes.offsets, st.routes.customers)
    return {"pairs": inst.granular_pairs, "full": _move(sol.eval()), "granular": _move(sol.eval(MASKS["granular"]))}


# --------------------------------------------------------------------- work --

def _evaluation(n, has_tw, pairs_per_row=None, per_pair=4, ops=7):
    """One evaluation: every distance once at 16 bits and the slot attributes, and a handful of integer
    operations per move (a pair of positions stands for about per_pair / 2 moves)."""
    q = n * 1.07
    pairs = q * (q if pairs_per_row is None else pairs_per_row) / 2
    return 2 * (pairs * 2) + q * (64 if has_tw else 32), pairs * per_pair * ops


def work(case):
    form = case["form"]
    if form in ("batch", "served"):
        steps = case["steps"] if form == "batch" else 4 * case["ticks"]
        one = [_evaluation(n, i % 2 == 1) for i, n in enumerate(_sizes(case))]
        return {"bytes": steps * sum(b for b, _ in one), "flops": steps * sum(f for _, f in one)}
    n, tw = case["n"], case["problem"] != "cvrp"
    if form == "query":
        b, f = _evaluation(n, tw)
        return {"bytes": b, "flops": f}
    if form == "setup":
        b, f = _evaluation(n, tw)
        g, h = _evaluation(n, tw, 1.2 * case["theta"])
        return {"bytes": 4 * (n + 1) ** 2 + 2 * (n + 1) ** 2 + 8 * n * case["theta"] + b + g, "flops": f + h + 2 * n * n}
    mode = case["mode"]
    b, f = _evaluation(n, tw, 1.2 * case["theta"] if mode == "granular" else None, 20 if mode == "variants" else 4)
    return {"bytes": case["steps"] * b, "flops": case["steps"] * f}


def exact(case, seed):
    """Every output is a whole number (moves, routes, costs, counts): there is no rounding to be told apart."""
    return None
