"""Applying a move on the device at the sizes where the step's forms change:
touched routes of 62..65 customers (a wavefront holds 63 and the depot), more
route slots than a workgroup has threads, and moved blocks of one and of
several rounds.  The routes and the cost are compared with the oracle's, and
every attribute through the best move and the move counts of a solution
freshly built from the same routes.  Integers throughout: equality."""
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


def move_id(sol, n, op, k, ra, pa, rb, pb):
    """Id of the move with refs at position pa of route ra and pb of rb (0: the start depot)."""
    Q = n + sol.R
    ref = lambda r, p: n + r if p == 0 else int(sol.customers[sol.offsets[r] + p - 1]) - 1  # noqa: E731
    a, b = ref(ra, pa), ref(rb, pb)
    if op in (1, 2, 3, 7, 8, 9) and a > b:
        a, b = b, a
        if op >= 7:
            op, k = 6 + k, op - 6
    return ((op * 4 + k) * Q + a) * Q + b


CASES = [
    # route lengths, then the moves (op, k, ra, pa, rb, pb) applied one after another
    ([63, 2, 62, 5], [(0, 1, 1, 1, 0, 63), (0, 1, 0, 64, 2, 0), (0, 1, 2, 10, 3, 2), (2, 0, 0, 30, 2, 31)]),
    ([64, 3, 1], [(0, 1, 0, 64, 2, 1), (2, 0, 0, 0, 1, 3), (4, 2, 1, 1, 1, 40), (3, 0, 1, 2, 1, 60)]),
    ([1, 7, 0, 9], [(0, 1, 0, 1, 2, 0), (1, 1, 1, 3, 3, 9), (2, 0, 0, 0, 3, 0), (1, 1, 1, 1, 1, 7)]),
    ([5] + [2] * 1300 + [6], [(0, 1, 0, 5, 1301, 6), (2, 0, 0, 1, 1301, 2), (0, 1, 1301, 1, 0, 0), (1, 1, 3, 1, 1200, 2)]),
    ([9] + [40] * 60 + [3], [(0, 1, 61, 2, 0, 3), (2, 0, 0, 2, 61, 1), (4, 3, 7, 1, 7, 30)]),
]
VARIANTS = [(5, 3, 0, 1, 1, 2), (6, 2, 1, 1, 0, 0), (8, 3, 0, 1, 1, 1)]


@pytest.mark.parametrize("form", ["plain", "general", "penalised"])
@pytest.mark.parametrize("problem", ["cvrp", "vrptw", "vrpspdtw"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_apply_forms(tga, case, problem, form):
    lengths, moves = CASES[case]
    if problem == "vrpspdtw" and form == "plain":
        pytest.skip("pickups are evaluated on the general path")
    inst, sol = make(problem, lengths, 900 + case)
    if form != "plain" and case in (0, 2):
        moves = moves + VARIANTS if case == 2 else moves + [(5, 3, 0, 1, 1, 1), (9, 1, 0, 2, 2, 3)]
    I = tga.Instance.from_workload(inst)

    def solution(s):
        S = tga.Solution(I, s.offsets, s.customers)
        if form == "general":
            S.set_general(True)
        elif form == "penalised":
            S.set_penalty(3, 0 if problem == "cvrp" else 2)
        return S

    S = solution(sol)
    for mv in moves:
        mid = move_id(sol, inst.n, *mv)
        m = tga.Move()
        m.op, m.k, m.id, m.version, m.feas = mv[0], mv[1], mid, S.version, 3
        print("apply", problem, form, mv, flush=True)
        cost = S.apply(m)
        sol = oracle.apply_move(inst, sol, mid)
        off, cust, c = S.get()
        assert np.array_equal(off, sol.offsets) and np.array_equal(cust, sol.customers)
        assert cost == c == oracle.cost(inst, sol)[0]
        F = solution(sol)
        a, b = S.eval(), F.eval()
        assert (a is None) == (b is None) and (a is None or (a.id, a.delta) == (b.id, b.delta))
        assert np.array_equal(S.move_counts(), F.move_counts())
        if form != "plain":
            assert S.violations() == F.violations()


@pytest.mark.parametrize("problem", ["cvrp", "vrptw", "vrpspdtw"])
@pytest.mark.parametrize("lengths", [[1], [0, 0, 3], [63] * 3, [63, 64, 1], [9] * 16, [9] * 17, [200, 3], [4, 0] * 40])
def test_set_reload_get(tga, problem, lengths):
    """Setting, reloading and reading back routes where the build changes form (one and several workgroups of 16
    routes, a route too long for a wavefront): evaluations and counts equal the oracle's for the routes given."""
    inst, sol = make(problem, lengths, 1200 + len(lengths))
    other = make(problem, lengths, 1300 + len(lengths))[1]
    S = tga.Solution(tga.Instance.from_workload(inst), sol.offsets, sol.customers)
    print("set / reload / get", problem, len(lengths), flush=True)
    for k, s in enumerate((sol, other, sol)):
        if k > 0:
            S.reload(s.offsets, s.customers)
        off, cust, cost = S.get()
        assert np.array_equal(off, s.offsets) and np.array_equal(cust, s.customers)
        assert cost == oracle.cost(inst, s)[0]
        ob = oracle.eval_neighbourhood(inst, s, 0x1F, threads=0)
        b = S.eval()
        assert (b is not None) == bool(ob.found) and (b is None or (b.id, b.delta) == (ob.id, ob.delta))
        assert int(S.move_counts().sum()) == ob.moves
        if problem == "vrpspdtw":
            assert S.violations() == oracle.violations(inst, s)
        if b is not None:
            S.apply(b)  # the next reload replaces changed routes


@pytest.mark.parametrize("lengths", [[12] * 9, [60, 62, 3, 5, 58, 1, 0], [2] * 300])
@pytest.mark.parametrize("problem", ["cvrp", "vrptw", "vrpspdtw"])
def test_multi_steps(tga, problem, lengths):
    """Multi-move steps: candidates kept in LDS and read from the table, routes that outgrow a wavefront."""
    inst, sol = make(problem, lengths, 1400 + len(lengths))
    S = tga.Solution(tga.Instance.from_workload(inst), sol.offsets, sol.customers)
    S.set_multi(True)
    print("multi", problem, len(lengths), flush=True)
    steps = 4
    fin, applied, per, evaluated = oracle.local_search_multi(inst, sol, 0x1F, max_steps=steps)
    got, moves, cost = S.ls_run(steps, 0x1F | tga.OP_MULTI)
    assert (got, moves) == (len(per), evaluated) and S.multi_stats() == (len(per), len(applied))
    off, cust, c = S.get()
    assert np.array_equal(off, fin.offsets) and np.array_equal(cust, fin.customers)
    assert cost == c == oracle.cost(inst, fin)[0]
    F = tga.Solution(S.inst, off, cust)
    F.set_general(True)
    a, b = S.eval(), F.eval()
    assert (a is None) == (b is None) and (a is None or (a.id, a.delta) == (b.id, b.delta))
    assert np.array_equal(S.move_counts(), F.move_counts()) and S.violations() == F.violations()
