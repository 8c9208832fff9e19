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
