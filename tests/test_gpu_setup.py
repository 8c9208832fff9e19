"""Registering an instance at the sizes where the check's tiles end, with a
fault planted in each corner of the matrix, and neighbour lists with ties,
one neighbour, every neighbour and the widest distances, against the oracle.
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


@pytest.mark.parametrize("has_tw", [0, 1])
@pytest.mark.parametrize("n", [1, 7, 62, 63, 64, 127, 128, 200])
def test_check_instance(tga, n, has_tw):
    inst = W.make_vrptw(n, 50 + n) if has_tw else W.make_cvrp(n, 50 + n)
    sol = W.sweep(inst)
    I = tga.Instance.from_workload(inst)
    assert I.dist_bytes == 2
    S = tga.Solution(I, sol.offsets, sol.customers)
    ob, b = oracle.eval_neighbourhood(inst, sol, 0x1F, threads=0), S.eval()
    assert (b is not None) == bool(ob.found) and (b is None or (b.id, b.delta) == (ob.id, ob.delta))

    def load(dist, node4):
        return tga.Instance(n, dist, node4, inst.capacity, has_tw)

    for i, j in {(0, n), (n, 0), (n, n // 2), (n // 2, n - 1), (n - 1, 0)}:
        if i == j:
            continue
        d = inst.dist.copy()
        d[i, j] += 1
        with pytest.raises(tga.TGAError, match="symmetric"):
            load(d, inst.node4)
        d[j, i] = d[i, j] = -1
        with pytest.raises(tga.TGAError, match="outside"):
            load(d, inst.node4)
        d[j, i] = d[i, j] = 1 << 24
        with pytest.raises(tga.TGAError, match="outside"):
            load(d, inst.node4)
        d[j, i] = d[i, j] = 65535
        assert load(d, inst.node4).dist_bytes == 2
        d[j, i] = d[i, j] = 65536
        assert load(d, inst.node4).dist_bytes == 4
    for i in (0, n // 2, n):
        d = inst.dist.copy()
        d[i, i] = 3
        with pytest.raises(tga.TGAError, match="diagonal"):
            load(d, inst.node4)
        for col, v in ((0, -1), (0, 1 << 26)) + (((1, -5), (3, -1), (2, 1 << 26)) if has_tw else ()):
            nd = inst.node4.copy()
            nd[i, col] = v
            with pytest.raises(tga.TGAError):
                load(inst.dist, nd)


def neighbours_case(kind, n):
    if kind == "ties":
        return W.tiny_instance(n, 70 + n, n % 2 == 0, dup=True, span=12)
    inst = W.make_cvrp(n, 80 + n)
    if kind == "equal":
        inst.dist = (np.ones((n + 1, n + 1), np.int32) - np.eye(n + 1, dtype=np.int32)) * 700
    elif kind == "widest":
        inst.dist = np.minimum(inst.dist * 15000, (1 << 24) - 1).astype(np.int32)
    return inst


@pytest.mark.parametrize("kind,n", [("ties", 40), ("ties", 257), ("equal", 130), ("widest", 50), ("plain", 300)])
@pytest.mark.parametrize("part", [0, 7, 2, 1])
def test_neighbour_lists(tga, kind, n, part):
    inst = neighbours_case(kind, n)
    theta = 1 if part == 0 else n // part
    sol = W.random_solution(inst, max(3, n // 9), 90 + n)
    print("neighbours", kind, n, theta, flush=True)
    I = tga.Instance.from_workload(inst)
    I.set_granular(theta)
    mask = oracle.granular_mask(inst, theta)
    assert I.granular_pairs == int(mask[1:, 1:].sum()) + int(mask[1:, 0].sum())
    S = tga.Solution(I, sol.offsets, sol.customers)
    fin, ids, deltas, moves = oracle.local_search(inst, sol, 0x1F, max_steps=6, theta=theta, mask=mask)
    steps, mv, _ = S.ls_run(6, 0x1F | tga.OP_GRANULAR)
    off, cust, _ = S.get()
    assert (steps, mv) == (len(ids), moves)
    assert np.array_equal(off, fin.offsets) and np.array_equal(cust, fin.customers)
