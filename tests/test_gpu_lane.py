"""GPU: one lane per operation (the default launch shape) at the edges of its
wavefronts, workgroups and lookahead, against the oracle: operation counts
around 64 and 256, tables filled to the last cell (probes that pass every
cell, runs that wrap), and mixed requests in rounds that end inside a
workgroup."""
import numpy as np
import pytest

import oracle
from paper_1601_04017_amd import inputs
from tests.gpu_util import keys_dtype, make_table, to_dev, to_host

pytestmark = pytest.mark.gpu

LAYOUTS = [oracle.PACKED32, oracle.KV64]


def _keys(layout, n, seed, absent=False):
    f = inputs.distinct_keys_u32 if layout == oracle.PACKED32 else inputs.distinct_keys_u64
    return f(n, seed, absent=absent)


@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("n", [1, 63, 64, 65, 255, 256, 257, 1000])
def test_every_operation(layout, n):
    dt = keys_dtype(layout)
    log2c = 11
    t, o = make_table(layout, log2c), oracle.OracleTable(layout, log2c)
    k = _keys(layout, n, 31 + n)
    v = np.arange(1, n + 1, dtype=dt)
    absent = _keys(layout, n, 31 + n, absent=True)
    k[0] = 1  # a reserved key among them
    both = np.concatenate([absent, k])
    bv = np.concatenate([v, v + dt(5)])
    assert np.array_equal(to_host(t.insert(to_dev(k), to_dev(v))), o.insert(k, v))
    assert np.array_equal(to_host(t.insert_or_update(to_dev(both), to_dev(bv), op=oracle.ASSIGN)),
                          o.insert_or_update(both, bv, oracle.ASSIGN))
    assert np.array_equal(to_host(t.update(to_dev(k), None, op=oracle.ADD)), o.update(k, None, oracle.ADD))
    gone = both[::3].copy()
    assert np.array_equal(to_host(t.erase(to_dev(gone))), o.erase(gone))
    gv, gf = t.find(to_dev(both))
    ov, of = o.find(both)
    assert np.array_equal(to_host(gf), of)
    assert np.array_equal(to_host(gv, dt), ov)
    assert t.count() == o.counts()
    assert t.status() == -4
    t.close()


@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("log2c", [6, 9])
def test_table_filled_to_the_last_cell(layout, log2c):
    dt = keys_dtype(layout)
    c = 1 << log2c
    t = make_table(layout, log2c)
    k = _keys(layout, c + 7, 77)
    v = np.arange(1, c + 8, dtype=dt)
    f = to_host(t.insert(to_dev(k), to_dev(v)))
    # which 7 find no cell is open; the rest are in
    assert (f == 1).sum() == c and (f == 0xFF).sum() == 7
    assert t.status() == -3
    assert t.count() == (c, c)
    gv, gf = t.find(to_dev(k))
    inside = f == 1
    assert np.array_equal(to_host(gf), inside.astype(np.uint8))
    assert np.array_equal(to_host(gv, dt), np.where(inside, v, 0))
    absent = _keys(layout, 300, 77, absent=True)
    gv, gf = t.find(to_dev(absent))
    assert not to_host(gf).any() and not to_host(gv).any()
    assert not to_host(t.update(to_dev(absent), None, op=oracle.ADD)).any()
    assert not to_host(t.erase(to_dev(absent))).any()
    up = to_host(t.insert_or_update(to_dev(np.concatenate([k[inside], absent])), None, op=oracle.ASSIGN))
    assert not up[:c].any() and (up[c:] == 0xFF).all()
    assert to_host(t.erase(to_dev(k[inside]))).all()
    assert t.count() == (c, 0)
    t.close()


@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("n", [1, 127, 128, 129, 700])
def test_mixed_requests_in_short_rounds(layout, n):
    from paper_1601_04017_amd import lpht
    torch = pytest.importorskip("torch")
    dt = keys_dtype(layout)
    rng = np.random.default_rng(n)
    tabs, want, ops, outs = [], [], [], []
    kinds_of = []
    for j in range(3):
        t, o = make_table(layout, 8 + j, auto_grow=True), oracle.OracleTable(layout, 8 + j, auto_grow=True)
        k = _keys(layout, n, 400 + j)
        o.insert(k[::2].copy(), None)
        t.insert(to_dev(k[::2].copy()), None)
        kinds = rng.choice(np.array([0, 1, 2], np.uint8), n)
        flags = torch.full((n,), 7, dtype=torch.uint8, device="cuda")
        vals = torch.full((n,), 7, dtype=torch.int32 if layout == oracle.PACKED32 else torch.int64, device="cuda")
        dk, dkinds = to_dev(k), to_dev(kinds)
        for op, up, sel in ((lpht.OP_FIND, 0, 0), (lpht.OP_UPSERT, lpht.ADD, 1), (lpht.OP_ERASE, 0, 2)):
            ops.append(dict(table=t, op=op, up=up, keys=dk, vals_out=vals if sel == 0 else None, flags=flags,
                            kinds=dkinds, kind_sel=sel, count_sel=int((kinds == sel).sum())))
        ov, of = o.find(k)
        flag = np.where(kinds == 0, of, 0).astype(np.uint8)
        flag[kinds == 1] = o.insert_or_update(k[kinds == 1], None, oracle.ADD)
        flag[kinds == 2] = o.erase(k[kinds == 2])
        tabs.append((t, o))
        outs.append((vals, flags))
        want.append((np.where(kinds == 0, ov, 0).astype(dt), flag, int((kinds == 0).sum())))
    b = lpht.Batch(16)
    b.run(ops)
    for (t, o), (vals, flags), (wv, wf, finds) in zip(tabs, outs, want):
        assert np.array_equal(to_host(flags), wf)
        if finds:
            assert np.array_equal(to_host(vals, dt), wv)
        assert t.count() == o.counts()
        t.close()
    b.close()
