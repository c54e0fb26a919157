"""GPU: request arrays at every alignment, pinned and pageable mixed, through
the serving waves, against the oracle: each request's slice of a buffer begins
at its own byte offset, with guard bytes on both sides that must stay."""
import numpy as np
import pytest

import oracle
from paper_1601_04017_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", [oracle.PACKED32, oracle.KV64])
@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("pinned", [True, False])
def test_unaligned_slices(layout, mode, pinned):
    import torch
    from paper_1601_04017_amd import lpht
    kdt = np.uint32 if layout == oracle.PACKED32 else np.uint64
    w = np.dtype(kdt).itemsize
    # sizes around the 16-byte pieces and the 16 KiB work items; more tables
    # than one launch's descriptors hold
    sizes = [1, 2, 3, 15, 16, 17, 31, 33, 129, 1000, 2047, 2049, 4097, 16385] + list(range(40, 76))
    rng = np.random.default_rng(5)
    ntab = len(sizes)
    srv = lpht.Server([10] * ntab, layout=layout, mode=mode, max_inflight=64, streams=2)
    total = sum(sizes) * 2 + 64

    def buf(nbytes, fill):
        t = torch.full((nbytes,), fill, dtype=torch.uint8)
        return t.pin_memory() if pinned else t

    keys, vals = buf((total + 2 * ntab) * w, 0xA5), buf((total + 2 * ntab) * w, 0xA5)
    kinds, flags = buf(total + 20 * ntab, 0xA5), buf(total + 20 * ntab, 0xA5)
    arr = (lpht.lpht_request * ntab)()
    spans, oracles = [], []
    ko = bo = 3
    for j, n in enumerate(sizes):
        f = inputs.distinct_keys_u32 if layout == oracle.PACKED32 else inputs.distinct_keys_u64
        k = f(n, 60 + j)
        kd = rng.choice(np.array([0, 1, 2], np.uint8), n)
        keys.numpy()[ko * w:(ko + n) * w] = k.view(np.uint8)
        kinds.numpy()[bo:bo + n] = kd
        arr[j] = lpht.lpht_request(j, 0, n, keys.data_ptr() + ko * w, kinds.data_ptr() + bo,
                                   vals.data_ptr() + ko * w, flags.data_ptr() + bo)
        spans.append((ko, bo, n, k, kd))
        oracles.append(oracle.OracleTable(layout, 10, auto_grow=True))
        ko += n + 1
        bo += n + 1 + j % 17
    for _ in range(2):  # the second pass finds what the first inserted
        srv.run_closed_loop(arr, 16)
        vb, fb = vals.numpy().copy(), flags.numpy().copy()
        for (k0, b0, n, k, kd), o in zip(spans, oracles):
            ov, of = o.find(k)
            want = np.where(kd == 0, of, 0).astype(np.uint8)
            want[kd == 1] = o.insert_or_update(k[kd == 1], None, oracle.ADD)
            want[kd == 2] = o.erase(k[kd == 2])
            assert np.array_equal(fb[b0:b0 + n], want)
            assert np.array_equal(vb[k0 * w:(k0 + n) * w].view(kdt), np.where(kd == 0, ov, 0).astype(kdt))
            fb[b0:b0 + n] = 0xA5
            vb[k0 * w:(k0 + n) * w] = 0xA5
        assert (fb == 0xA5).all() and (vb == 0xA5).all(), "bytes outside the requests were written"
    for j, o in enumerate(oracles):
        assert srv.table(j).count() == o.counts()
    srv.close()
