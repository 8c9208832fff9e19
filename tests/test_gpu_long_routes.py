"""Solutions that hold routes longer than a wavefront (64 positions) or than
what a workgroup stages: the forms taken for them, compared with the oracle.
Integers throughout: equality."""
import numpy as np
import pytest

import oracle
from paper_2506_17357_amd import workload as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tga():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2506_17357_amd import tga as T
    T.lib()
    return T


def make(problem, lengths, seed):
    n = int(sum(lengths))
    kw = dict(demand_max=9, capacity=10 ** 6)
    inst = {"cvrp": W.make_cvrp, "vrptw": W.make_vrptw, "vrpspdtw": W.make_vrpspdtw}[problem](n, seed, **kw)
    perm = np.random.Generator(np.random.PCG64(seed)).permutation(np.arange(1, n + 1)).astype(np.int32)
    return inst, W.Solution(np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32), perm)


def fields(m):
    return None if m is None else (m.op, m.k, m.a, m.b, m.delta, m.id)


@pytest.mark.parametrize("problem", ["cvrp", "vrptw", "vrpspdtw"])
@pytest.mark.parametrize("lengths", [[64, 2], [1, 0, 700, 64, 3, 900], [63, 64, 65] * 8, [1030]])
def test_static_long_routes(tga, problem, lengths):
    """The entry point without a workspace, where the routes are staged in the arrays the build writes."""
    inst, sol = make(problem, lengths, 1500 + len(lengths))
    I = tga.Instance.from_workload(inst)
    print("static", problem, len(lengths), sum(lengths), flush=True)
    ob = oracle.eval_neighbourhood(inst, sol, 0x1F, threads=0)
    want = (ob.delta, ob.id) if ob.found else None
    other = make(problem, [5] * 9, 1600)
    for _ in range(2):
        m = tga.eval_routes_static(I, sol.offsets, sol.customers)
        assert (None if m is None else (m.delta, m.id)) == want
        assert fields(m) == fields(tga.Solution(I, sol.offsets, sol.customers).eval())
        # another instance's call in between overwrites the scratch
        tga.eval_routes_static(tga.Instance.from_workload(other[0]), other[1].offsets, other[1].customers)


def seconds(f, reps=15):
    """Median time of a call that waits for the device, after one to warm up."""
    import time

    import torch
    f()
    times = []
    for _ in range(reps):
        torch.cuda.synchronize()
        t = time.perf_counter()
        f()
        torch.cuda.synchronize()
        times.append(time.perf_counter() - t)
    return sorted(times)[reps // 2]


def spread(n, R):
    return [n // R + (i < n % R) for i in range(R)]


@pytest.mark.parametrize("form", ["plain", "general"])
@pytest.mark.parametrize("problem", ["cvrp", "vrptw", "vrpspdtw"])
@pytest.mark.parametrize("lengths", [[9] * 15 + [64] + [9] * 20, [64] * 17, [0] * 20 + [300] + [5] * 30, [1100, 0, 1]])
def test_reload_long_among_short(tga, problem, lengths, form):
    """A workgroup's share of the routes with a long one in it, beside workgroups that have none."""
    inst, sol = make(problem, lengths, 1700 + len(lengths))
    other = make(problem, lengths[::-1], 1800 + len(lengths))[1]
    S = tga.Solution(tga.Instance.from_workload(inst), sol.offsets, sol.customers)
    if form == "general":
        S.set_general(True)
    general = form == "general" or problem == "vrpspdtw"
    print("reload", problem, form, len(lengths), flush=True)
    for s in (other, sol):
        S.reload(s.offsets, s.customers)
        off, cust, cost = S.get()
        assert np.array_equal(off, s.offsets) and np.array_equal(cust, s.customers)
        assert cost == oracle.cost(inst, s)[0]
        for mask in (0x1F, 0xFF) if general else (0x1F,):
            ob = oracle.eval_neighbourhood(inst, s, mask, threads=0)
            b = S.eval(mask)
            assert (b is not None) == bool(ob.found) and (b is None or (b.id, b.delta) == (ob.id, ob.delta))
        assert int(S.move_counts().sum()) == oracle.eval_neighbourhood(inst, s, 0x1F, threads=0).moves
        if general:
            assert S.violations() == oracle.violations(inst, s)


def test_reload_time_with_one_long_route(tga):
    """One route of 64 customers among 500 short ones: the short ones are built as without it (about as fast;
    4 times as long when every slot of the solution went through one workgroup)."""
    times = []
    for lengths in (spread(10000, 500), [64] + spread(9936, 499)):
        inst, sol = make("cvrp", lengths, 1900)
        S = tga.Solution(tga.Instance.from_workload(inst), sol.offsets, sol.customers)
        times.append(seconds(lambda: S.reload(sol.offsets, sol.customers)))
    print("reload, all short and one of 64: %.1f %.1f us" % (times[0] * 1e6, times[1] * 1e6), flush=True)
    assert times[1] < 2 * times[0]


@pytest.mark.parametrize("lengths", [[9] * 20 + [90] + [8] * 9, [200, 3, 0, 150, 64], [63, 62, 61, 60] * 5, [70]])
@pytest.mark.parametrize("problem", ["cvrp", "vrptw", "vrpspdtw"])
def test_multi_steps_long(tga, problem, lengths):
    """Multi-move steps with long routes that moves touch and leave alone, in one and in several workgroups."""
    inst, sol = make(problem, lengths, 2000 + len(lengths))
    S = tga.Solution(tga.Instance.from_workload(inst), sol.offsets, sol.customers)
    S.set_multi(True)
    print("multi", problem, len(lengths), flush=True)
    fin, applied, per, evaluated = oracle.local_search_multi(inst, sol, 0x1F, max_steps=5)
    got, moves, cost = S.ls_run(5, 0x1F | tga.OP_MULTI)
    assert (got, moves) == (len(per), evaluated) and S.multi_stats() == (len(per), len(applied))
    off, cust, c = S.get()
    assert np.array_equal(off, fin.offsets) and np.array_equal(cust, fin.customers)
    assert cost == c == oracle.cost(inst, fin)[0]
    F = tga.Solution(S.inst, off, cust)
    F.set_general(True)
    assert fields(S.eval()) == fields(F.eval())
    assert np.array_equal(S.move_counts(), F.move_counts()) and S.violations() == F.violations()


def test_multi_time_with_one_long_route(tga):
    """A multi-move step lays every route out once, a long one among them or not (2 to 3 times as long with one of
    100; 20 times when every selected move was applied by itself)."""
    times = []
    for lengths in (spread(1000, 60), [100] + spread(900, 59)):
        inst, sol = make("cvrp", lengths, 2100)
        S = tga.Solution(tga.Instance.from_workload(inst), sol.offsets, sol.customers)
        S.set_multi(True)

        def run():
            S.reload(sol.offsets, sol.customers)
            assert S.ls_run(6, 0x1F | tga.OP_MULTI)[0] == 6
        times.append(seconds(run, reps=7))
    print("6 multi-move steps, all short and one of 100: %.0f %.0f us" % (times[0] * 1e6, times[1] * 1e6), flush=True)
    assert times[1] < 6 * times[0]


@pytest.mark.parametrize("problem", ["cvrp", "vrptw", "vrpspdtw"])
@pytest.mark.parametrize("lengths", [[64], [63, 128, 1, 127, 0, 129], [5] * 30 + [190, 66] + [4] * 7])
def test_summaries_of_long_routes(tga, problem, lengths):
    """Every move of the general path, which reads the summaries of every slot: after switching it on, after a reload
    and after moves into, out of and within long routes."""
    inst, sol = make(problem, lengths, 2200 + len(lengths))
    I = tga.Instance.from_workload(inst)
    S = tga.Solution(I, sol.offsets, sol.customers)
    pen = (3, 0 if problem == "cvrp" else 2)
    print("summaries", problem, len(lengths), flush=True)

    def check(s, what):
        ob, odd, odf = oracle.eval_neighbourhood(inst, s, 0xFF, dump=True, threads=0, penalty=pen)
        gb, gdd, gdf = S.eval(0xFF, dump=True)
        assert np.array_equal(gdf.cpu().numpy(), odf) and np.array_equal(gdd.cpu().numpy(), odd), what
        assert (gb.delta, gb.id) == (ob.delta, ob.id)
        assert S.violations() == oracle.violations(inst, s), what

    S.set_penalty(*pen)
    check(sol, "switched on")
    S.reload(sol.offsets, sol.customers)
    check(sol, "reloaded")
    for k in range(3):
        # the best move under other weights, so that the three are of different kinds
        m = S.eval((0x1F, 0x60, 0x84)[k])
        if m is None:
            continue
        S.apply(m)
        sol = oracle.apply_move(inst, sol, m.id)
        check(sol, "applied %d" % k)


def test_summaries_time(tga):
    """Switching the general path on: routes of 70 customers in tiles of a wavefront, as fast as routes of 60 (25
    times as long with one thread per route)."""
    times = []
    for lengths in ([60] * 117, [70] * 100):
        inst, sol = make("vrptw", lengths, 2300)
        S = tga.Solution(tga.Instance.from_workload(inst), sol.offsets, sol.customers)
        times.append(seconds(lambda: S.set_general(True)))
    print("set_general, routes of 60 and of 70: %.1f %.1f us" % (times[0] * 1e6, times[1] * 1e6), flush=True)
    assert times[1] < 4 * times[0]


@pytest.mark.parametrize("form", ["plain", "penalised"])
@pytest.mark.parametrize("problem", ["cvrp", "vrptw", "vrpspdtw"])
def test_totals_after_moves_on_long_routes(tga, problem, form):
    """Cost, violations and move counts after moves that lengthen, shorten, empty and rearrange long routes, one
    after another, against a solution set from the same routes."""
    if problem == "vrpspdtw" and form == "plain":
        pytest.skip("pickups are evaluated on the general path")
    inst, sol = make(problem, [130, 3, 64, 200, 0], 2400)
    I = tga.Instance.from_workload(inst)

    def solution(s):
        S = tga.Solution(I, s.offsets, s.customers)
        if form == "penalised":
            S.set_penalty(3, 0 if problem == "cvrp" else 2)
        return S

    S = solution(sol)
    Q = inst.n + sol.R
    rng = np.random.Generator(np.random.PCG64(2400))
    done = 0
    print("totals", problem, form, flush=True)
    while done < 30:
        op = int(rng.integers(0, 5)) if form == "plain" else int(rng.integers(0, 10))
        k = {0: 1, 1: 1, 2: 0, 3: 0}.get(op, int(rng.integers(1, 4)))
        a, b = sorted(rng.integers(0, Q, size=2).tolist()) if op in (1, 2, 3, 7, 8, 9) else rng.integers(0, Q, size=2).tolist()
        m = tga.Move()
        m.op, m.k, m.id, m.version, m.feas = op, k, ((op * 4 + k) * Q + a) * Q + b, S.version, 3
        try:
            cost = S.apply(m)
        except tga.TGAError:
            continue  # not a move of these routes
        done += 1
        sol = oracle.apply_move(inst, sol, m.id)
        F = solution(sol)
        assert cost == oracle.cost(inst, sol)[0]
        assert np.array_equal(S.move_counts(), F.move_counts()), (op, k, a, b)
        if form != "plain":
            assert S.violations() == F.violations() == oracle.violations(inst, sol), (op, k, a, b)
        assert fields(S.eval()) == fields(F.eval())


def test_multi_selection_beyond_the_lds(tga):
    """A selection of more moves than a step keeps decoded is applied move by move: routes, cost and counts."""
    inst, sol = make("cvrp", [2] * 1500, 2500)
    S = tga.Solution(tga.Instance.from_workload(inst), sol.offsets, sol.customers)
    S.set_multi(True)
    print("multi, 1500 routes", flush=True)
    fin, applied, per, evaluated = oracle.local_search_multi(inst, sol, 0x1F, max_steps=1)
    assert len(applied) > 700
    got, moves, cost = S.ls_run(1, 0x1F | tga.OP_MULTI)
    assert (got, moves) == (len(per), evaluated) and S.multi_stats() == (len(per), len(applied))
    off, cust, c = S.get()
    assert np.array_equal(off, fin.offsets) and np.array_equal(cust, fin.customers)
    assert cost == c == oracle.cost(inst, fin)[0]
    F = tga.Solution(S.inst, off, cust)
    assert np.array_equal(S.move_counts(), F.move_counts())


WALKS = [[200, 3], [70, 0, 55, 64, 30], [17] * 6 + [0] * 90, [12, 0, 13, 0, 11, 0, 9] * 5 + [0] * 60, [52], [48, 1], [120]]


@pytest.mark.parametrize("mode", ["hard", "penalised"])
@pytest.mark.parametrize("problem", ["cvrp", "vrptw", "vrpspdtw"])
@pytest.mark.parametrize("case", range(len(WALKS)))
def test_general_walks(tga, case, problem, mode):
    """Intra-route moves on the general path of routes that are staged in a group, in turn, and not at all (too long,
    or too many to a group beside empty ones): every move, the best move, and steps."""
    inst, sol = make(problem, WALKS[case], 2600 + case)
    pen = None if mode == "hard" else (3, 0 if problem == "cvrp" else 2)
    S = tga.Solution(tga.Instance.from_workload(inst), sol.offsets, sol.customers)
    S.set_general(True) if pen is None else S.set_penalty(*pen)
    print("walks", problem, mode, case, flush=True)
    for mask in (0x1F, 0x18, 0x02):
        ob, odd, odf = oracle.eval_neighbourhood(inst, sol, mask, dump=True, threads=0, penalty=pen)
        gb, gdd, gdf = S.eval(mask, dump=True)
        assert np.array_equal(gdf.cpu().numpy(), odf) and np.array_equal(gdd.cpu().numpy(), odd)
        for b in (gb, S.eval(mask)):
            assert (b is not None) == bool(ob.found) and (b is None or (b.delta, b.id) == (ob.delta, ob.id))
    fin, ids, _, moves = oracle.local_search(inst, sol, 0x1F, max_steps=12, penalty=pen)
    steps, mv, _ = S.ls_run(12, 0x1F)
    off, cust, _ = S.get()
    assert (steps, mv) == (len(ids), moves)
    assert np.array_equal(off, fin.offsets) and np.array_equal(cust, fin.customers)


def test_general_walks_time(tga):
    """One route of 1000 customers: the general path spreads its first positions over the chip, the plain path (where
    a route is one workgroup's) is its measure: an eighth of it, and longer than it when they were one workgroup's."""
    inst, sol = make("cvrp", [1000], 2700)
    S = tga.Solution(tga.Instance.from_workload(inst), sol.offsets, sol.customers)

    def run():
        S.reload(sol.offsets, sol.customers)
        assert S.ls_run(3)[0] == 3
    times = [seconds(run, reps=5)]
    S.set_penalty(10)
    times.append(seconds(run, reps=5))
    print("3 steps, plain and penalised: %.0f %.0f us" % (times[0] * 1e6, times[1] * 1e6), flush=True)
    assert times[1] < 0.5 * times[0]
