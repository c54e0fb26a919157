"""GPU: blocks of the library's memory cache going from one table to another
while their last use is still queued: on the same stream at once, on another
stream only when it has completed, from several threads; and everything given
back by lpht_release_pools."""
import threading

import numpy as np
import pytest

from paper_1601_04017_amd import inputs
from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


def _grow_and_check(seed, stream, n=60_000, passes=6):
    """Tables that grow (old cells freed behind the migration that reads them)
    and go, one after the other without a wait, then every key is looked up."""
    import torch
    from paper_1601_04017_amd import lpht
    with torch.cuda.stream(stream):
        k = inputs.distinct_keys_u64(n, seed)
        dk, dv = to_dev(k), to_dev(np.arange(n, dtype=np.uint64))
        got = []
        for _ in range(passes):
            t = lpht.Table(log2_capacity=12, auto_grow=True, stream=stream)
            for lo in range(0, n, 7_001):
                t.insert(dk[lo:lo + 7_001], dv[lo:lo + 7_001], flags=False, stream=stream)
            got.append(t.find(dk, stream=stream))
            t.close()
        stream.synchronize()
    for v, f in got:
        assert to_host(f).all()
        assert np.array_equal(to_host(v, np.uint64), np.arange(n, dtype=np.uint64))


def test_same_stream():
    import torch
    _grow_and_check(1, torch.cuda.current_stream())


def test_streams_in_turn():
    import torch
    for j in range(4):
        _grow_and_check(10 + j, torch.cuda.Stream(), passes=2)


def test_threads_with_streams_of_their_own():
    import torch
    errors = []

    def work(j):
        try:
            _grow_and_check(20 + j, torch.cuda.Stream(), passes=4)
        except BaseException as e:  # noqa: BLE001 - reported below
            errors.append(e)

    threads = [threading.Thread(target=work, args=(j,)) for j in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors


def test_release_gives_everything_back():
    import torch
    from paper_1601_04017_amd import lpht
    import gc
    gc.collect()
    t = lpht.Table(log2_capacity=26)
    assert lpht.load().lpht_release_pools() == lpht.ERR_INVALID  # in use
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    t.close()
    if lpht.load().lpht_release_pools() == lpht.OK:  # (another test's objects may still be alive)
        assert torch.cuda.mem_get_info()[0] >= before + (16 << 26)
    # a new table makes a new pool
    t = lpht.Table(log2_capacity=12)
    k = to_dev(inputs.distinct_keys_u64(1000, 3))
    assert to_host(t.insert(k)).all()
    t.close()
