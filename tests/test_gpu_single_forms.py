"""The single-solution evaluation at the sizes where its forms change: routes
of 38..41 customers (what one staged region holds), groups that do not share
one, long and empty routes, strips with a remainder, and operator masks that
enable one kind of move only.  Every delta, feasibility bit and the best move
against the oracle.  Integers throughout: equality."""
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
    inst = {"cvrp": W.make_cvrp, "vrptw": W.make_vrptw, "vrpspdtw": W.make_vrpspdtw}[problem](
        n, seed, demand_max=9, capacity=max(20, 5 * n // len(lengths)))
    perm = np.random.Generator(np.random.PCG64(seed)).permutation(np.arange(1, n + 1)).astype(np.int32)
    return inst, W.Solution(np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32), perm)


LENGTHS = [[38, 39, 40, 41], [16, 17, 15, 16, 0, 1], [70, 3, 0, 5], [1] * 9, [8, 7, 9, 8, 8, 9, 7, 8, 13]]


def compare(T, S, inst, sol, mask, pen=None):
    ob, odd, odf = oracle.eval_neighbourhood(inst, sol, mask, dump=True, threads=0, penalty=pen)
    gb, gdd, gdf = S.eval(mask, dump=True)
    for got, want in ((gdf.cpu().numpy(), odf), (gdd.cpu().numpy(), odd)):
        bad = np.nonzero(got != want)[0]
        assert bad.size == 0, (bad.size, [(oracle.decode(S.Q, int(i)), int(want[i]), int(got[i])) for i in bad[:12]])
    for b in (gb, S.eval(mask)):  # with the dump every move is evaluated, without it the screens decide
        assert (b is not None) == bool(ob.found)
        assert b is None or (b.delta, b.id) == (ob.delta, ob.id)


@pytest.mark.parametrize("mask", [0x1F, 0x07, 0x18, 0x02])
@pytest.mark.parametrize("problem", ["cvrp", "vrptw"])
@pytest.mark.parametrize("case", range(len(LENGTHS)))
def test_plain_forms(tga, case, problem, mask):
    print("plain", problem, LENGTHS[case], hex(mask), flush=True)
    inst, sol = make(problem, LENGTHS[case], 300 + case)
    S = tga.Solution(tga.Instance.from_workload(inst), sol.offsets, sol.customers)
    for rows in (0, 1, 5):
        S.set_rows(rows)
        compare(tga, S, inst, sol, mask)


def widen(inst):
    """The instance with distances (and times) beyond 16 bits."""
    inst.dist = np.ascontiguousarray(inst.dist * 100)
    inst.node4 = inst.node4.copy()
    if inst.has_tw:
        inst.node4[:, 1:] *= 100
    assert inst.dist.max() >= 1 << 16
    return inst


@pytest.mark.parametrize("mode", ["hard", "penalised", "heavy"])
@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("problem", ["cvrp", "vrptw", "vrpspdtw"])
@pytest.mark.parametrize("case", range(len(LENGTHS)))
def test_general_forms(tga, case, problem, wide, mode):
    print("general", problem, LENGTHS[case], "wide" if wide else "", mode, flush=True)
    inst, sol = make(problem, LENGTHS[case], 400 + case)
    if wide:
        inst = widen(inst)
    S = tga.Solution(tga.Instance.from_workload(inst), sol.offsets, sol.customers)
    assert S.inst.dist_bytes == (4 if wide else 2)
    # light penalties, where most moves are screened, and ones that outweigh every distance
    pen = None if mode == "hard" else ((1, 1) if mode == "penalised" else (40, 3))
    if pen is not None:
        pen = (pen[0], 0 if problem == "cvrp" else (1 if wide else pen[1]))
    if pen is None:
        S.set_general(True)
    else:
        S.set_penalty(*pen)
    for mask in (0xFF, 0x1F, 0x60 if case % 2 else 0x82, 0x05):
        compare(tga, S, inst, sol, mask, pen)


@pytest.mark.parametrize("problem", ["cvrp", "vrptw", "vrpspdtw"])
def test_general_steps(tga, problem):
    """Local-search steps on the general path (screens from 0 on), all operators, against the oracle's."""
    inst, sol = make(problem, [13, 2, 9, 11, 0, 12, 10, 8, 14, 21], 500)
    for pen in (None, (2, 0) if problem == "cvrp" else (2, 3)):
        S = tga.Solution(tga.Instance.from_workload(inst), sol.offsets, sol.customers)
        S.set_general(True) if pen is None else S.set_penalty(*pen)
        fin, ids, deltas, moves = oracle.local_search(inst, sol, 0xFF, max_steps=25, penalty=pen)
        steps, mv, _ = S.ls_run(25, 0xFF)
        off, cust, _ = S.get()
        assert (steps, mv) == (len(ids), moves)
        assert np.array_equal(off, fin.offsets) and np.array_equal(cust, fin.customers)


@pytest.mark.parametrize("queued", [False, True])
def test_record_on_several_streams(tga, queued):
    """Evaluations and moves in turn on three streams, each behind a queue of other work that outlasts the
    short wait for the record or behind none."""
    import torch
    print("streams", "queued" if queued else "idle", flush=True)
    inst, sol = make("vrptw", [13, 2, 9, 11, 0, 12, 10, 8, 14, 21], 600)
    S = tga.Solution(tga.Instance.from_workload(inst), sol.offsets, sol.customers)
    final, ids, _, _ = oracle.local_search(inst, sol, max_steps=6)
    streams = [torch.cuda.Stream() for _ in range(3)]
    work = torch.zeros(1 << 26, device="cuda")  # 256 MiB: a pass takes about 0.1 ms
    torch.cuda.synchronize()
    for k, want in enumerate(ids):
        st = streams[k % 3]
        if queued:
            with torch.cuda.stream(st):
                for _ in range(8):
                    work.add_(1.0)
        best = S.eval(0x1F, stream=st)
        assert best is not None and best.id == want
        again = S.eval(0x1F, stream=streams[(k + 1) % 3])
        assert (again.delta, again.id) == (best.delta, best.id)
        S.apply(best, stream=streams[(k + 2) % 3])
    off, cust, cost = S.get()
    assert np.array_equal(off, final.offsets) and np.array_equal(cust, final.customers)
    assert cost == oracle.cost(inst, final)[0]
    torch.cuda.synchronize()
