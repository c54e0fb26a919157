"""The partitioned insert-or-add where its scatter's tiles end or are uneven:
the smallest call that is partitioned and ragged ones, a batch of one key
(every wavefront in one bucket, all other buckets empty), of two keys in
turn, of distinct keys, and of the reserved key alone; sums against exact
integer counts and flags by key."""
import numpy as np
import pytest

import oracle
from paper_1601_04017_amd import inputs, lpht
from tests.gpu_util import keys_dtype, make_table, to_dev, to_host

pytestmark = pytest.mark.gpu

MIN = 1 << 22  # smallest partitioned call


def _keys(what, layout, n):
    dt = keys_dtype(layout)
    if what == "distinct":
        return (inputs.distinct_keys_u64 if layout == oracle.KV64 else inputs.distinct_keys_u32)(n, 91).astype(dt)
    if what == "one":
        return np.full(n, 77, dt)
    if what == "two":
        return np.where(np.arange(n) % 2 == 0, 5, 1_000_003).astype(dt)
    if what == "reserved":
        return np.zeros(n, dt)
    z = inputs.scramble_keys_u64(inputs.zipf_keys_u64(n, n, 1.1, seed=92), 93).astype(dt)
    return np.maximum(z, dt(2))


@pytest.mark.parametrize("layout", [oracle.PACKED32, oracle.KV64])
@pytest.mark.parametrize("what,n,mul", [("one", MIN, 0), ("two", MIN + 1, 0), ("reserved", MIN, 0),
                                        ("distinct", MIN + 4095, 0), ("zipf", MIN + 63, 0),
                                        ("zipf", MIN + 4097, 0x9E3779B97F4A7C15)])
@pytest.mark.parametrize("form", ["plain", "vals", "flags", "both"])
def test_tiles(layout, what, n, mul, form):
    z = _keys(what, layout, n)
    v = (np.arange(n) % 5 + 1).astype(keys_dtype(layout)) if form in ("vals", "both") else None
    flags = form in ("flags", "both")
    t = make_table(layout, 23, **({"hash": lpht.HASH_MULSHIFT, "mul": mul} if mul else {}))
    # into an empty table, then into one that holds the keys
    for turn in (1, 2):
        f = t.insert_or_update(to_dev(z), None if v is None else to_dev(v), op=oracle.ADD, flags=flags)
        if what == "reserved":
            if flags:
                assert (to_host(f) == 0xFE).all()
            assert t.count() == (0, 0)
            assert t.status() == lpht.ERR_RESERVED_KEY
            continue
        uniq, inv = np.unique(z, return_inverse=True)
        if flags:
            f = to_host(f)
            assert ((f == 0) | (f == 1)).all()
            per_key = np.bincount(inv, weights=f, minlength=uniq.size)
            assert (per_key == (1 if turn == 1 else 0)).all()
        if turn == 1:
            got, found = t.find(to_dev(uniq))
            want = np.bincount(inv, weights=None if v is None else v, minlength=uniq.size).astype(np.uint64)
            assert to_host(found).all()
            assert np.array_equal(to_host(got, keys_dtype(layout)).astype(np.uint64), want)
        assert t.count() == (uniq.size, uniq.size)
        assert t.status() == 0
        if n + uniq.size > 1 << 23:  # (a second turn could find the table full)
            break
