"""Calls that fail after their launches: what they leave on the device must not
reach the results of later calls.  Integers throughout: equality."""
import ctypes

import pytest

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


def plant_error(T):
    """Leave an error of an earlier runtime call of this thread (a device that does not exist) to be found."""
    hip = T.lib()  # the library's own runtime symbols
    hip.hipSetDevice.restype = ctypes.c_int
    hip.hipSetDevice.argtypes = [ctypes.c_int]
    assert hip.hipSetDevice(9999) != 0


@pytest.mark.parametrize("call", ["eval", "get", "reload"])
def test_failed_call_leaves_nothing_in_flight(tga, call):
    import torch
    print("failed call", call, flush=True)
    made = [(i, W.sweep(i)) for i in (W.make_vrptw(150, 21), W.make_cvrp(150, 22))]
    one, two = (tga.Solution(tga.Instance.from_workload(i), s.offsets, s.customers) for i, s in made)
    want = two.eval()
    first = (want.delta, want.id)
    busy, free = torch.cuda.Stream(), torch.cuda.Stream()
    work = torch.zeros(1 << 26, device="cuda")  # 256 MiB: a pass takes about 0.1 ms
    torch.cuda.synchronize()
    with torch.cuda.stream(busy):
        for _ in range(20):
            work.add_(1.0)
    plant_error(tga)
    with pytest.raises(tga.TGAError):
        if call == "eval":
            one.eval(stream=busy)
        elif call == "get":
            one.get(stream=busy)
        else:
            one.reload(made[0][1].offsets, made[0][1].customers, stream=busy)
    assert busy.query()  # the call came back with its work done
    for _ in range(100):
        m = two.eval(stream=free)
        assert (m.delta, m.id) == first
    torch.cuda.synchronize()
    again = one.eval()
    fresh = tga.Solution(one.inst, made[0][1].offsets, made[0][1].customers).eval()
    assert (again.delta, again.id) == (fresh.delta, fresh.id)
