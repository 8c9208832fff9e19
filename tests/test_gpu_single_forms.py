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
    assert np.array_equal(gdf.cpu().numpy(), odf)
    assert np.array_equal(gdd.cpu().numpy(), odd)
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
