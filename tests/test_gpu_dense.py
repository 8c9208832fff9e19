"""The general path where the screens let most moves through (windows and
capacities broken on every route, ties of many empty routes, dumps): a
wavefront then takes its remaining steps with every move in place.  Every move
and the best move against the oracle.  Integers throughout: equality."""
import time

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


def make(problem, lengths, seed, **kw):
    n = int(sum(lengths))
    inst = {"cvrp": W.make_cvrp, "vrptw": W.make_vrptw, "vrpspdtw": W.make_vrpspdtw}[problem](n, seed, **kw)
    perm = np.random.Generator(np.random.PCG64(seed)).permutation(np.arange(1, n + 1)).astype(np.int32)
    return inst, W.Solution(np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32), perm)


LENGTHS = [[17] * 24 + [0] * 250, [13, 16, 1, 2, 20, 3] * 8, [5] * 100]


@pytest.mark.parametrize("mode", ["hard", "penalised", "multi"])
@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("problem", ["cvrp", "vrptw", "vrpspdtw"])
@pytest.mark.parametrize("case", range(len(LENGTHS)))
def test_dense_steps(tga, case, problem, wide, mode):
    inst, sol = make(problem, LENGTHS[case], 3100 + case, demand_max=30, capacity=150)
    if wide:  # distances (and times) beyond 16 bits
        inst.dist = np.ascontiguousarray(inst.dist * 60)
        if inst.has_tw:
            inst.node4[:, 1:] *= 60
        assert inst.dist.max() >= 1 << 16
    print("dense", problem, case, "wide" if wide else "", mode, flush=True)
    S = tga.Solution(tga.Instance.from_workload(inst), sol.offsets, sol.customers)
    if mode == "multi":
        S.set_multi(True)
        fin, applied, per, evaluated = oracle.local_search_multi(inst, sol, 0x1F, max_steps=2)
        got, moves, cost = S.ls_run(2, 0x1F | tga.OP_MULTI)
        assert (got, moves) == (len(per), evaluated) and S.multi_stats() == (len(per), len(applied))
        off, cust, _ = S.get()
        assert np.array_equal(off, fin.offsets) and np.array_equal(cust, fin.customers)
        return
    pen = None
    if mode == "penalised":
        # weights under which the routes' excess outweighs the distances, as far as the scores' range lets them
        pen = (1, 0) if wide else (5, 0 if problem == "cvrp" else 10)
        S.set_penalty(*pen)
    else:
        S.set_general(True)
    for mask in (0xFF, 0x1F, 0x81, 0x66):
        ob, odd, odf = oracle.eval_neighbourhood(inst, sol, mask, dump=True, threads=0, penalty=pen)
        gb, gdd, gdf = S.eval(mask, dump=True)
        for got, want in ((gdf.cpu().numpy(), odf), (gdd.cpu().numpy(), odd)):
            bad = np.nonzero(got != want)[0]
            assert bad.size == 0, (hex(mask), bad.size, [(oracle.decode(S.Q, int(i)), int(want[i]), int(got[i])) for i in bad[:8]])
        for b in (gb, S.eval(mask)):
            assert (b is not None) == bool(ob.found) and (b is None or (b.delta, b.id) == (ob.delta, ob.id)), hex(mask)
    fin, ids, _, moves = oracle.local_search(inst, sol, 0xFF, max_steps=4, penalty=pen)
    steps, mv, _ = S.ls_run(4, 0xFF)
    off, cust, _ = S.get()
    assert (steps, mv) == (len(ids), moves)
    assert np.array_equal(off, fin.offsets) and np.array_equal(cust, fin.customers)


def test_spare_vehicles_time(tga):
    """60 routes with broken windows and 2000 spare vehicles: a penalised step takes about as long as the plain path's
    evaluation of the same routes (4 times as long when every move that passed the screens was a queue entry)."""
    import torch
    inst = W.make_vrptw(1000, 1077, capacity=10 ** 6)
    order = np.asarray(W._angle_order(inst), np.int32)
    lengths = [17] * 40 + [16] * 20 + [0] * 2000
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    S = tga.Solution(tga.Instance.from_workload(inst), off, order)

    def median(f):
        return sorted(f() for _ in range(7))[3]

    def plain():
        t = time.perf_counter()
        S.eval()
        return time.perf_counter() - t

    def step():
        S.reload(off, order)
        torch.cuda.synchronize()
        t = time.perf_counter()
        assert S.ls_run(15)[0] == 15
        return (time.perf_counter() - t) / 15
    times = [median(plain)]
    S.set_penalty(10, 10)
    times.append(median(step))
    print("plain evaluation, penalised step: %.0f %.0f us" % (times[0] * 1e6, times[1] * 1e6), flush=True)
    assert times[1] < 2 * times[0]
