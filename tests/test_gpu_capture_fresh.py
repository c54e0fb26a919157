"""Calls that load an empty table by region write its cells without reading
them: a table that a replayed graph fills (the host's counts know nothing of
replays), or whose clear was only captured, keeps what it holds."""
import pytest

import oracle
from paper_1601_04017_amd import inputs
from tests.gpu_util import make_table, to_dev

pytestmark = pytest.mark.gpu

N = 1 << 22


def _second_call(t, keys, how):
    if how == "insert":
        t.insert(keys, None, flags=False)
    else:
        t.insert_or_update(keys, None, op=oracle.ADD, flags=False)


@pytest.mark.parametrize("how", ["insert", "add"])
@pytest.mark.parametrize("captured", ["insert", "clear"])
def test_eager_call_keeps_what_a_replay_inserted(captured, how):
    import torch
    allk = to_dev(inputs.distinct_keys_u64(N + 5000, 98))
    a, b = allk[:5000].contiguous(), allk[5000:].contiguous()
    t = make_table(oracle.KV64, 24)
    g = torch.cuda.CUDAGraph()
    if captured == "clear":
        t.insert(a, None, flags=False)
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        t.insert(a, None, flags=False) if captured == "insert" else t.clear()
    if captured == "insert":
        assert t.count() == (0, 0)
        g.replay()
        torch.cuda.synchronize()
    _second_call(t, b, how)
    assert t.count() == (N + 5000, N + 5000)
    assert bool(t.find(allk)[1].all())
    t.clear()
    t.insert(a, None, flags=False)
    if captured == "clear":
        for _ in range(3):
            g.replay()
            assert t.count() == (0, 0)
            t.insert(a, None, flags=False)
    assert t.count() == (5000, 5000)
