"""GPU: inserting calls on string tables longer than one slice of their two
launches, with keys that come again in the same slice and in the next one, and
a workgroup's worth around its edges: values, flags and counts against sums."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SLICE = 1 << 20


@pytest.mark.parametrize("n", [1023, 1024, 1025, SLICE - 1, SLICE + 5])
@pytest.mark.parametrize("upsert", [False, True])
def test_keys_again_within_and_across_slices(n, upsert):
    import torch
    from paper_1601_04017_amd import lpht
    rng = np.random.default_rng(n)
    number = rng.integers(0, max(1, n // 3), n).astype(np.uint64)
    # lengths 8 to 11: the number, then up to three fixed bytes told by it
    length = 8 + (number % 4).astype(np.int64)
    offs = np.zeros(n + 1, dtype=np.int64)
    offs[1:] = np.cumsum(length)
    raw = np.full(int(offs[-1]), 0x5A, dtype=np.uint8)
    view = number.view(np.uint8).reshape(-1, 8)
    for b in range(8):
        raw[offs[:-1] + b] = view[:, b]
    vals = rng.integers(1, 1000, n).astype(np.uint64)
    L, p = lpht._str_lib(), lpht._ptr
    dbytes, doffs = torch.from_numpy(raw).cuda(), torch.from_numpy(offs).cuda()
    dvals = torch.from_numpy(vals.view(np.int64)).cuda()
    flags = torch.full((n,), 9, dtype=torch.uint8, device="cuda")
    t = lpht.StrTable(log2_capacity=10, auto_grow=True, pool_bytes=4096)
    stream = lpht._stream_handle(None)
    if upsert:
        rc = L.lpht_str_insert_or_update(t._h, p(dbytes), p(doffs), n, p(dvals), lpht.ADD, p(flags), stream)
    else:
        rc = L.lpht_str_insert(t._h, p(dbytes), p(doffs), n, p(dvals), p(flags), stream)
    assert rc == lpht.OK and t.status() == 0
    f = flags.cpu().numpy()
    u, where = np.unique(number, return_inverse=True)
    # exactly one operation of each key inserted it
    assert set(np.unique(f)) <= {0, 1}
    assert np.array_equal(np.bincount(where, weights=f, minlength=u.size), np.ones(u.size))
    assert t.count() == (u.size, u.size)
    got = torch.zeros(n, dtype=torch.int64, device="cuda")
    found = torch.zeros(n, dtype=torch.uint8, device="cuda")
    assert L.lpht_str_find(t._h, p(dbytes), p(doffs), n, p(got), p(found), stream) == lpht.OK
    assert found.cpu().numpy().all()
    g = got.cpu().numpy().view(np.uint64)
    if upsert:
        sums = np.zeros(u.size, dtype=np.uint64)
        np.add.at(sums, where, vals)
        assert np.array_equal(g, sums[where])
    else:
        winner = np.zeros(u.size, dtype=np.uint64)
        winner[where[f == 1]] = vals[f == 1]
        assert np.array_equal(g, winner[where])
    t.close()
