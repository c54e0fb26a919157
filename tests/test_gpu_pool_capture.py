"""GPU: the library's memory cache while another stream is captured in the
global mode (tables made, resized, loaded through scratch and closed by the same
and by another thread, none of it part of the capture), and everything given
back by lpht_release_pools in a process whose only table is closed."""
import os
import subprocess
import sys
import threading

import numpy as np
import pytest

from paper_1601_04017_amd import inputs
from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu

N = (1 << 20) + 3


@pytest.mark.parametrize("elsewhere", ["thread", "stream"])
def test_allocations_beside_a_capture(elsewhere):
    import torch
    from paper_1601_04017_amd import lpht
    k, v = inputs.distinct_keys_u64(N, 5), np.arange(N, dtype=np.uint64)
    dk, dv = to_dev(k), to_dev(v)
    x = torch.arange(1000, device="cuda")
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    # blocks in the cache whose last use was on a third stream
    c = torch.cuda.Stream()
    lpht.Table(log2_capacity=21, stream=c).close(c)
    lpht.Table(log2_capacity=12, stream=c).close(c)
    torch.cuda.synchronize()
    # made in advance: torch's own allocations are not what is tested
    found = torch.zeros(N, dtype=torch.uint8, device="cuda")
    got = torch.zeros(N, dtype=torch.int64, device="cuda")
    errors = []

    def work():
        try:
            for lg in (12, 20, 22):  # the first two resized before the load
                t = lpht.Table(log2_capacity=lg, auto_grow=True, stream=b)
                t.insert(dk, dv, flags=False, stream=b)
                t.find(dk, got, found, stream=b)
                t.close(b)
        except BaseException as e:  # noqa: BLE001 - reported below
            errors.append(e)

    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=a, capture_error_mode="global"):
        y = x * 3
        if elsewhere == "thread":
            th = threading.Thread(target=work)
            th.start()
            th.join()
        else:
            work()
        z = y + 1
    assert not errors, errors
    b.synchronize()
    assert to_host(found).all() and np.array_equal(to_host(got, np.uint64), v)
    for j in range(3):
        x.add_(j)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(z, x * 3 + 1)


def test_release_returns_the_memory():
    code = """
import torch
from paper_1601_04017_amd import lpht
torch.zeros(1, device="cuda")
torch.cuda.synchronize()
before = torch.cuda.mem_get_info()[0]
t = lpht.Table(log2_capacity=26)
torch.cuda.synchronize()
assert torch.cuda.mem_get_info()[0] <= before - (16 << 26)
t.close()
assert lpht.load().lpht_release_pools() == lpht.OK
assert torch.cuda.mem_get_info()[0] >= before - (64 << 20), (before, torch.cuda.mem_get_info()[0])
"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    p = subprocess.run([sys.executable, "-c", code], cwd=root, capture_output=True, text=True, timeout=110)
    assert p.returncode == 0, p.stderr
