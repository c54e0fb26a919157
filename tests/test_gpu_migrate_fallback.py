"""GPU: migrations of tables filled beyond two thirds, where clusters longer than
a block's halo are regular and the whole move is done again by cluster: every key
keeps its value, and the move takes a small multiple of the block migration's
time."""
import numpy as np
import pytest

from paper_1601_04017_amd import inputs
from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("to", [0, 1])
def test_keys_survive(to):
    from paper_1601_04017_amd import lpht
    n = int(0.74 * (1 << 20))
    k = inputs.distinct_keys_u64(n, 6)
    t = lpht.Table(log2_capacity=20, alpha=(9, 10))
    t.insert(to_dev(k), to_dev(np.arange(n, dtype=np.uint64)), flags=False)
    t.erase(to_dev(k[::3]), flags=False)
    t.grow(20 + to)
    got, found = t.find(to_dev(k))
    assert np.array_equal(to_host(found) == 0, np.arange(n) % 3 == 0)
    keep = np.arange(n) % 3 != 0
    assert np.array_equal(to_host(got, np.uint64)[keep], np.arange(n, dtype=np.uint64)[keep])
    assert t.count() == (keep.sum(), keep.sum())
    t.close()


def test_time_of_a_full_table():
    # 24 times with a quarter of the workgroups, 11.5 with all
    import torch
    from paper_1601_04017_amd import lpht
    lg = 26
    k = to_dev(inputs.distinct_keys_u64(int(0.74 * (1 << lg)), 1))

    def best(fill):
        ms = []
        for _ in range(3):
            t = lpht.Table(log2_capacity=lg, alpha=(9, 10))
            t.insert(k[:int(fill * (1 << lg))], None, flags=False)
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            t.grow(lg)
            b.record()
            torch.cuda.synchronize()
            ms.append(a.elapsed_time(b))
            t.close()
        return min(ms)

    assert best(0.74) < 17 * best(0.5)
