"""GPU: calls in which reserved keys are frequent: every one of them has its flag,
the sticky error is set, and the call takes about the time of one without."""
import numpy as np
import pytest

from paper_1601_04017_amd import inputs
from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


def test_time_and_flags():
    import torch
    from paper_1601_04017_amd import lpht
    n = 1 << 22
    k = inputs.distinct_keys_u64(1000, 2)[np.random.default_rng(1).integers(0, 1000, n)]
    bad = k.copy()
    where = np.random.default_rng(2).random(n) < 0.03
    bad[where] = np.arange(where.sum()) % 2
    t = lpht.Table(log2_capacity=16)
    t.insert(to_dev(k), None)

    def best(keys):
        ms = []
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            got = t.find(keys)[1]
            b.record()
            torch.cuda.synchronize()
            ms.append(a.elapsed_time(b))
        return min(ms), to_host(got)

    base, f = best(to_dev(k))
    assert f.all() and t.status() == 0
    ms, f = best(to_dev(bad))
    assert np.array_equal(f, np.where(where, 0xFE, 1)) and t.status() == lpht.ERR_RESERVED_KEY
    assert ms < 4 * base
    t.close()
