"""Insert-or-add of a large batch into an empty table, whose buckets own their
regions: regions filled so far that many keys run past their end and are put
off, alone and with sums (2^22 operations on 2^22 cells, 15/16 full), and
buckets of more keys than a workgroup has slots for; against the oracle's
table, or exact sums by key and absent keys not found."""
import numpy as np
import pytest

import oracle
from paper_1601_04017_amd import inputs
from tests import helpers as H
from tests.gpu_util import cells_host, make_table, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("with_vals", [False, True])
@pytest.mark.parametrize("distinct", [15, 8, 5])  # sixteenths of the operations
def test_regions_run_over(with_vals, distinct):
    n = 1 << 22
    base = inputs.distinct_keys_u64(n * distinct // 16, 95)
    z = np.resize(base, n)[inputs.permutation(n, 96)]
    v = (np.arange(n) % 7 + 1).astype(np.uint64) if with_vals else None
    t = make_table(oracle.KV64, 22)
    t.insert_or_update(to_dev(z), None if v is None else to_dev(v), op=oracle.ADD, flags=False)
    o = oracle.OracleTable(oracle.KV64, 22)
    o.insert_or_update(z, v, oracle.ADD)
    assert t.count() == o.counts()
    assert t.status() == 0
    H.assert_same_table_modulo_run_order(cells_host(t), o.cells(), oracle.KV64)


@pytest.mark.parametrize("with_vals", [False, True])
def test_more_keys_than_slots(with_vals):
    n = 3 << 24  # 6144 keys a bucket
    import torch
    z = to_dev(inputs.distinct_keys_u64(n, 97))
    v = torch.arange(1, n + 1, dtype=torch.int64, device="cuda") if with_vals else None
    t = make_table(oracle.KV64, 26)
    t.insert_or_update(z, v, op=oracle.ADD, flags=False)
    assert t.count() == (n, n)
    assert t.status() == 0
    got, found = t.find(z)
    assert bool(found.all())
    assert bool((got == (v if with_vals else 1)).all())
    absent = to_dev(inputs.distinct_keys_u64(1 << 20, 97, absent=True))
    assert not bool(t.find(absent)[1].any())
