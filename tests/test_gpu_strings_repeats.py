"""GPU: inserting calls on string tables whose absent keys come many times: the
pool takes one record for each key that is inserted, and no more."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _call(t, kind, number, vals):
    import torch
    from paper_1601_04017_amd import lpht
    L, p = lpht._str_lib(), lpht._ptr
    n = number.size
    length = 8 + (number % 29).astype(np.int64)
    offs = np.zeros(n + 1, dtype=np.int64)
    offs[1:] = np.cumsum(length)
    raw = np.full(int(offs[-1]), 0x33, dtype=np.uint8)
    view = number.astype(np.uint64).view(np.uint8).reshape(-1, 8)
    for b in range(8):
        raw[offs[:-1] + b] = view[:, b]
    keep = [torch.from_numpy(raw).cuda(), torch.from_numpy(offs).cuda(), torch.from_numpy(vals.view(np.int64)).cuda()]
    flags = torch.full((n,), 9, dtype=torch.uint8, device="cuda")
    out = torch.zeros(n, dtype=torch.int64, device="cuda")
    st = lpht._stream_handle(None)
    a = (t._h, p(keep[0]), p(keep[1]), n)
    rc = {"insert": lambda: L.lpht_str_insert(*a, p(keep[2]), p(flags), st),
          "assign": lambda: L.lpht_str_insert_or_update(*a, p(keep[2]), lpht.ASSIGN, p(flags), st),
          "add": lambda: L.lpht_str_insert_or_update(*a, p(keep[2]), lpht.ADD, p(flags), st),
          "find": lambda: L.lpht_str_find(*a, p(out), p(flags), st)}[kind]()
    assert rc == lpht.OK
    return flags.cpu().numpy(), out.cpu().numpy().view(np.uint64)


def _records(number):
    """Bytes of the distinct keys' records: length word and key, in whole words."""
    u = np.unique(number)
    return int(((4 + 8 + u % 29 + 7) // 8 * 8).sum())


@pytest.mark.parametrize("kind", ["insert", "assign", "add"])
@pytest.mark.parametrize("n,distinct", [(2000, 1), (70_000, 3), (300_000, 1000), ((1 << 20) + 77, 200_000)])
def test_one_record_per_inserted_key(kind, n, distinct):
    from paper_1601_04017_amd import lpht
    rng = np.random.default_rng(distinct)
    number = rng.integers(0, distinct, n)
    vals = rng.integers(1, 1 << 40, n).astype(np.uint64)
    t = lpht.StrTable(log2_capacity=20, pool_bytes=1 << 26)
    f, _ = _call(t, kind, number, vals)
    u, where = np.unique(number, return_inverse=True)
    assert np.array_equal(np.bincount(where, weights=f, minlength=u.size), np.ones(u.size)) and f.max() == 1
    assert t.count() == (u.size, u.size) and t.status() == 0
    assert t.capacity()[1] == 8 + _records(number)  # (records start at 8)
    found, got = _call(t, "find", number, vals)
    assert found.all()
    if kind == "add":
        sums = np.zeros(u.size, dtype=np.uint64)
        np.add.at(sums, where, vals)
        assert np.array_equal(got, sums[where])
    elif kind == "insert":
        winner = np.zeros(u.size, dtype=np.uint64)
        winner[where[f == 1]] = vals[f == 1]
        assert np.array_equal(got, winner[where])
    else:
        # some operation's value, the same for all operations of the key
        order = np.lexsort((vals, where))
        pairs = set(zip(where[order].tolist(), vals[order].tolist()))
        assert all(x in pairs for x in zip(where.tolist(), got.tolist()))
    # the same again, with new keys among them: only those take records
    more = np.concatenate([number[:1000], np.arange(distinct, distinct + 5), np.arange(distinct, distinct + 5)])
    f, _ = _call(t, kind, more, np.ones(more.size, dtype=np.uint64))
    assert f.sum() == 5
    assert t.capacity()[1] == 8 + _records(np.concatenate([number, more]))
    t.close()


def test_full_table_and_keys_it_holds():
    # no cell left: absent keys are refused, their flags say so, no record stays
    from paper_1601_04017_amd import lpht
    t = lpht.StrTable(log2_capacity=6, pool_bytes=1 << 20)
    number = np.arange(100)
    f, _ = _call(t, "insert", np.concatenate([number, number]), np.ones(200, dtype=np.uint64))
    assert (f == 1).sum() == 64 and t.status() == lpht.ERR_FULL
    held = number[(f[:100] == 1) | (f[100:] == 1)]
    assert t.capacity()[1] == 8 + _records(held)
    assert np.array_equal(f.reshape(2, 100).max(axis=0) == 0xFF, ~np.isin(number, held))
    t.close()
