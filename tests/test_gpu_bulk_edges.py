"""GPU: sort-based build and merge where their passes change: element counts
around a tile, some cell of a block with a few or many copies, and a batch
just below and above the skew that takes the combining passes; cell for cell
against the oracle."""
import numpy as np
import pytest

import oracle
from paper_1601_04017_amd import inputs
from tests.gpu_util import cells_host, keys_dtype, make_table, to_dev

pytestmark = pytest.mark.gpu

LAYOUTS = [oracle.PACKED32, oracle.KV64]


def _keys(layout, n, seed):
    f = inputs.distinct_keys_u32 if layout == oracle.PACKED32 else inputs.distinct_keys_u64
    return f(n, seed)


def _check(layout, log2c, batches, op):
    t, o = make_table(layout, log2c), oracle.OracleTable(layout, log2c)
    for j, (k, v) in enumerate(batches):
        (t.build if j == 0 else t.merge)(to_dev(k), to_dev(v), op=op)
        (o.build if j == 0 else o.merge)(k, v, op)
        assert np.array_equal(cells_host(t), o.cells())
        assert t.count() == o.counts()
    t.close()


@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("n", [1, 4095, 4096, 4097, 8191, 8193])
def test_around_a_tile(layout, n):
    dt = keys_dtype(layout)
    k = _keys(layout, n + 70, 5 + n)
    v = np.arange(n + 70, dtype=dt)
    _check(layout, 15, [(k[:n], v[:n]), (k[n // 2:], v[n // 2:] + dt(9))], oracle.ASSIGN)


@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("op", [oracle.ASSIGN, oracle.ADD])
@pytest.mark.parametrize("copies", [2, 11, 12, 13, 14, 200, 254, 255, 256, 257, 1025])
def test_copies_of_one_key(layout, op, copies):
    dt = keys_dtype(layout)
    rng = np.random.default_rng(copies)
    k = _keys(layout, 30_000, 9)
    k = np.concatenate([k, np.repeat(k[77], copies - 1)])[rng.permutation(30_000 + copies - 1)]
    _check(layout, 17, [(k, rng.integers(0, 1 << 20, k.size).astype(dt))], op)


@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("share", [0.01, 0.02, 0.3])
def test_around_the_skew(layout, share):
    # 256 bins: one key with 2.5, 5 and 76 times a bin's share of the batch
    dt = keys_dtype(layout)
    rng = np.random.default_rng(int(share * 100))
    n = 900_000
    k = _keys(layout, n, 21)
    k[rng.random(n) < share] = k[0]
    _check(layout, 22, [(k, rng.integers(0, 1 << 20, n).astype(dt))], oracle.ADD)
