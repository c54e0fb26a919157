"""GPU: loading a nearly empty table region by region, against the oracle, at
the calls where its passes differ: one partition level and two, the smallest
call, with and without flags and values, a table with elements, tombstones and
erased cells, equal keys that overflow their buckets, keys crowded at a
region's end, reserved keys, and sampled batches with and without common
keys."""
import numpy as np
import pytest

import oracle
from paper_1601_04017_amd import inputs
from tests import helpers as H
from tests.gpu_util import cells_host, keys_dtype, to_dev, to_host

pytestmark = pytest.mark.gpu

LAYOUTS = [oracle.PACKED32, oracle.KV64]
N0 = 1 << 20  # the smallest call


def _keys(layout, n, seed, absent=False):
    f = inputs.distinct_keys_u32 if layout == oracle.PACKED32 else inputs.distinct_keys_u64
    return f(n, seed, absent=absent)


def _pair(layout, log2c, **kw):
    from paper_1601_04017_amd import lpht
    okw = dict(kw)
    if kw.get("hash"):
        okw.pop("hash")
    return lpht.Table(layout=layout, log2_capacity=log2c, **kw), oracle.OracleTable(layout, log2c, **okw)


def _same(t, o, layout, log2c):
    assert t.count() == o.counts()
    cells = cells_host(t)
    H.assert_same_table_modulo_run_order(cells, o.cells(), layout)


@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("n,log2c", [(N0, 21), (N0 + 1, 21), (1_200_000, 21), (1_500_001, 22), ((1 << 22) + 1, 24)])
@pytest.mark.parametrize("flags", [True, False])
def test_distinct_keys_into_an_empty_table(layout, n, log2c, flags):
    dt = keys_dtype(layout)
    t, o = _pair(layout, log2c)
    k, v = _keys(layout, n, n % 1000 + 1), np.arange(n, dtype=dt)
    of = o.insert(k, v)
    gf = t.insert(to_dev(k), to_dev(v), flags=flags)
    if flags:
        assert np.array_equal(to_host(gf), of)
    assert t.status() == 0
    _same(t, o, layout, log2c)
    t.close()


@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("op", ["insert", "assign"])
def test_elements_and_tombstones_already_there(layout, op):
    # 2 * 10^5 elements, half of them erased, then 1.12 * 10^6 operations, some on
    # live keys, some on erased ones, some reserved
    dt = keys_dtype(layout)
    log2c = 21
    t, o = _pair(layout, log2c)
    k0 = _keys(layout, 200_000, 5)
    t.insert(to_dev(k0), None)
    o.insert(k0, None)
    t.erase(to_dev(k0[::2].copy()))
    o.erase(k0[::2].copy())
    t.count()  # (the host's bound on used cells becomes exact)
    k = _keys(layout, 1_120_000, 6)
    k[1::3] = np.resize(k0, k[1::3].size)[:k[1::3].size]
    k[0] = 0
    k[100_000] = 1
    k = np.concatenate([k[:100], k])  # the first hundred twice
    v = np.arange(7, 7 + k.size, dtype=dt)
    if op == "insert":
        gf, of = to_host(t.insert(to_dev(k), to_dev(v))), o.insert(k, v)
    else:
        gf = to_host(t.insert_or_update(to_dev(k), to_dev(v), op=oracle.ASSIGN))
        of = o.insert_or_update(k, v, oracle.ASSIGN)
    assert np.array_equal(H.canonical_flags(k, gf), H.canonical_flags(k, of))
    assert t.status() == -4
    assert t.count() == o.counts()
    # values: of a key that came several times, one of its operations' (or the
    # table's, for insert)
    gv, gfound = t.find(to_dev(k))
    ov, ofound = o.find(k)
    assert np.array_equal(to_host(gfound), ofound)
    gv = to_host(gv, dt)
    u, first, counts = np.unique(k, return_index=True, return_counts=True)
    once = first[counts == 1]
    assert np.array_equal(gv[once], ov[once])
    for key in u[counts > 1][:2000]:
        if key < 2:
            continue
        where = np.flatnonzero(k == key)
        stored = ov[where[0]]
        assert gv[where[0]] in set(v[where].tolist()) | {int(stored)}
    H.check_invariants(cells_host(t), layout, log2c)
    ko, kg = H.key_run_starts(o.cells(), layout)[0], H.key_run_starts(cells_host(t), layout)[0]
    assert np.array_equal(ko, kg)
    t.close()


@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("distinct", [1, 10, 3000, 100_000])
def test_equal_keys(layout, distinct):
    # far more operations per bucket than its room, or many copies in each
    dt = keys_dtype(layout)
    n, log2c = 1_400_001, 21
    rng = np.random.default_rng(distinct)
    base = _keys(layout, distinct, 8)
    k = base[rng.integers(0, distinct, n)]
    v = np.arange(n, dtype=dt)
    t, o = _pair(layout, log2c)
    gf, of = to_host(t.insert(to_dev(k), to_dev(v))), o.insert(k, v)
    assert np.array_equal(H.canonical_flags(k, gf), of)
    assert t.count() == o.counts()
    d = H.live_dict(cells_host(t), layout)
    for i in np.flatnonzero(gf == 1)[:3000]:
        assert d[int(k[i])] == int(v[i])
    _, ofound = o.find(base)
    assert np.array_equal(to_host(t.find(to_dev(base))[1]), ofound)
    H.check_invariants(cells_host(t), layout, log2c)
    t.close()


def test_keys_crowded_at_the_end_of_regions():
    # multiplier 1: the position is the key's top bits; runs of keys at the last
    # cells of regions go on in the next region, and past the table's end
    from paper_1601_04017_amd import lpht
    log2c, n = 21, N0 + 5
    rng = np.random.default_rng(3)
    c = 1 << log2c
    pos = rng.integers(0, c, n).astype(np.uint64)
    crowd = rng.random(n) < 0.1
    pos[crowd] = (rng.integers(1, c // 4096 + 1, crowd.sum()).astype(np.uint64) * np.uint64(4096)) - np.uint64(1)
    k = (pos << np.uint64(64 - log2c)) | rng.permutation(n).astype(np.uint64) + np.uint64(2)
    v = np.arange(n, dtype=np.uint64)
    t = lpht.Table(layout=lpht.KV64, log2_capacity=log2c, hash=lpht.HASH_MULSHIFT, mul=1)
    f = to_host(t.insert(to_dev(k), to_dev(v)))
    assert f.all() and t.count() == (n, n) and t.status() == 0
    gv, gf = t.find(to_dev(k))
    assert to_host(gf).all() and np.array_equal(to_host(gv, np.uint64), v)
    # every key reachable from its home: the cells between are not empty
    cells = cells_host(t)
    occ = cells[0::2] != 0
    at = np.flatnonzero(occ)
    home = (cells[0::2][at] >> np.uint64(64 - log2c)).astype(np.int64)
    empties = np.concatenate([[0], np.cumsum(~occ)])
    lo, hi = home, at
    wraps = hi < lo
    between = np.where(wraps, empties[c] - empties[lo] + empties[hi], empties[np.maximum(hi, lo)] - empties[lo])
    assert not between.any()
    absent = k ^ np.uint64(1 << 40)
    absent = absent[~np.isin(absent, k)][:100_000]
    assert not to_host(t.find(to_dev(absent))[1]).any()
    t.close()


@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("skew", [False, True])
def test_sampled_batches(layout, skew):
    dt = keys_dtype(layout)
    n, log2c = (1 << 22) + 3, 23
    if skew:
        k = inputs.zipf_keys_u64(n, 1_000_000, 1.0, seed=9).astype(dt)
    else:
        k = _keys(layout, n, 11)
    v = (np.arange(n) % 1000).astype(dt)
    t, o = _pair(layout, log2c)
    gf, of = to_host(t.insert(to_dev(k), to_dev(v))), o.insert(k, v)
    assert np.array_equal(H.canonical_flags(k, gf), of)
    assert t.count() == o.counts() and t.status() == 0
    u = np.unique(k)
    assert to_host(t.find(to_dev(u))[1]).all()
    assert not to_host(t.find(to_dev(_keys(layout, 100_000, 11, absent=True)))[1]).any() or skew
    t.close()
