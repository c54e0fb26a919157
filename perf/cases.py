"""The table operations whose speed is watched, at the sizes they are used at.

Each case is one pass of a program over the library's public entry points: the
loads, lookups, counts, growing loads, deletion windows, bulk builds, string
keys and served requests of the test suite and the benchmark, from a table that
fits one workgroup's share of a cache to the 2^28-cell table of the headline
benchmark.  `listed()` names twelve of them, `draw()` gives others of the same
ranges, `prepare()` makes what a program holds before the pass (keys, values,
resident tables), `run()` is the pass, `work()` what it cannot do without and
`exact()` its results by sorting and indexing alone.
"""
import math

import numpy as np
import torch

from paper_1601_04017_amd import lpht

#: The launch shape the autotuner picks on this GPU for large KV64 tables; a
#: program that autotunes runs with it, others with the library's defaults.
TUNED = dict(block_threads=512, group_width=1, blocks_per_cu=8, migrate_block=256, aggregate=1,
             g_find=(1, 1, 4, 8), g_modify=(2, 2, 4, 8))

#: One multiplier for the tables that hash by multiplication.
MUL = 0x9E3779B97F4A7C15


def listed():
    return [
        # a small dictionary rebuilt and looked up: latency and launches
        dict(name="load_find_tiny", kind="load_find", layout="kv64", log2_capacity=12, n=1500, flags=True,
             tuned=False, hash="crc"),
        # the packed benchmark size: 2^20 operations on 2^21 cells of 8 bytes
        dict(name="load_find_packed_1m", kind="load_find", layout="packed32", log2_capacity=21, n=1 << 20,
             flags=True, tuned=False, hash="crc"),
        # the headline benchmark's load and lookups, in its tuned launch shape
        dict(name="load_find_kv64_100m", kind="load_find", layout="kv64", log2_capacity=28, n=10 ** 8,
             flags=False, tuned=True, hash="crc"),
        # every modifying operation on one table, odd sizes, flags wanted
        dict(name="modify_kv64_3m", kind="modify", layout="kv64", log2_capacity=23, n=3_000_001, hash="crc"),
        # a request's worth of lookups on a resident table: the ordinary call
        dict(name="lookup_300k_in_16m", kind="lookup", layout="kv64", log2_capacity=24, stored=6_000_000,
             n=300_007, hash="crc"),
        # word-count style aggregation of a skewed stream (Zipf 1.0)
        dict(name="count_zipf_100m", kind="count", layout="kv64", log2_capacity=28, n=10 ** 8, s=1.0,
             universe=10 ** 8, tuned=True),
        # a table growing from 4096 cells under batches of 2^20
        dict(name="growing_20m", kind="growing", layout="kv64", n=20_000_000, batch=1 << 20),
        # one call of unknown distinct count, the table growing inside the kernel
        dict(name="growing_in_kernel_10m", kind="in_kernel", layout="kv64", n=10_000_000, s=1.0,
             universe=10 ** 8),
        # a sliding window: insert the next batch, erase the oldest one
        dict(name="window_1m", kind="window", layout="kv64", log2_capacity=21, window=1_000_000,
             batch=1 << 16, steps=24),
        # sort-based bulk build and merge of a further batch
        dict(name="bulk_10m", kind="bulk", layout="kv64", log2_capacity=25, n=10_000_000, m=1_000_003),
        # byte-string keys of 8 to 40 bytes
        dict(name="strings_2m", kind="strings", log2_capacity=23, n=2_000_003),
        # requests served over many resident tables from pinned host memory
        dict(name="serving_96", kind="serving", tables=16, requests=96, median=16384, clients=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["load_find", "load_find", "modify", "lookup", "count", "growing", "in_kernel", "window",
                       "bulk", "strings", "serving"])
    layout = rng.choice(["kv64", "kv64", "packed32"])
    c = dict(kind=kind)
    if kind == "load_find":
        n = _log_int(rng, 100, 5 * 10 ** 7)
        c.update(layout=layout, n=n, log2_capacity=_capacity_for(n, rng.uniform(0.2, 0.7)),
                 flags=rng.random() < 0.5, tuned=rng.random() < 0.5, hash=rng.choice(["crc", "crc", "mul"]))
    elif kind == "modify":
        n = _log_int(rng, 1000, 10 ** 7)
        c.update(layout=layout, n=n, log2_capacity=_capacity_for(n, rng.uniform(0.2, 0.55)),
                 hash=rng.choice(["crc", "crc", "mul"]))
    elif kind == "lookup":
        stored = _log_int(rng, 1000, 3 * 10 ** 7)
        c.update(layout=layout, stored=stored, n=_log_int(rng, 50, 10 ** 7),
                 log2_capacity=_capacity_for(stored, rng.uniform(0.2, 0.75)), hash=rng.choice(["crc", "crc", "mul"]))
    elif kind == "count":
        n = _log_int(rng, 10 ** 4, 5 * 10 ** 7)
        c.update(layout="kv64", n=n, s=round(rng.uniform(0.5, 1.5), 2), universe=max(1000, 2 * n),
                 log2_capacity=_capacity_for(n, 0.5), tuned=rng.random() < 0.5)
    elif kind == "growing":
        n = _log_int(rng, 10 ** 5, 3 * 10 ** 7)
        c.update(layout=layout, n=n, batch=max(n // 40 + 1, _log_int(rng, 1 << 12, 1 << 21)))
    elif kind == "in_kernel":
        n = _log_int(rng, 10 ** 5, 3 * 10 ** 7)
        c.update(layout="kv64", n=n, s=round(rng.uniform(0.5, 1.5), 2), universe=10 ** 8)
    elif kind == "window":
        w = _log_int(rng, 2 * 10 ** 4, 5 * 10 ** 6)
        c.update(layout=layout, window=w, log2_capacity=_capacity_for(w, 0.5), batch=max(257, w // rng.randint(5, 40)),
                 steps=rng.randint(8, 28))
    elif kind == "bulk":
        n = _log_int(rng, 10 ** 4, 2 * 10 ** 7)
        c.update(layout=layout, n=n, m=max(1, n // rng.randint(2, 20)),
                 log2_capacity=_capacity_for(2 * n, rng.uniform(0.3, 0.8)))
    elif kind == "strings":
        n = _log_int(rng, 1000, 4 * 10 ** 6)
        c.update(n=n, log2_capacity=_capacity_for(n, rng.uniform(0.2, 0.5)))
    else:
        c.update(tables=rng.randint(4, 32), requests=rng.randint(16, 128), median=_log_int(rng, 2048, 30000),
                 clients=rng.choice([8, 32, 64, 128]))
    return c


def _capacity_for(n, fill):
    return max(10, min(27, math.ceil(math.log2(n / fill))))


# ---------------------------------------------------------------- inputs

def _dev():
    return torch.device("cuda")


def _signed(x):
    x &= (1 << 64) - 1
    return x - (1 << 64) if x >> 63 else x


def _shr(x, k):
    return (x >> k) & ((1 << (64 - k)) - 1)


def _mix64(x):
    """A bijection of the 64-bit integers (SplitMix64's output function)."""
    x = (x ^ _shr(x, 30)) * _signed(0xBF58476D1CE4E5B9)
    x = (x ^ _shr(x, 27)) * _signed(0x94D049BB133111EB)
    return x ^ _shr(x, 31)


def _mix32(x):
    """A bijection of the 32-bit integers (MurmurHash3's finaliser)."""
    m = 0xFFFFFFFF
    x = x ^ (x >> 16)
    x = (x * 0x85EBCA6B) & m
    x = x ^ (x >> 13)
    x = (x * 0xC2B2AE35) & m
    return x ^ (x >> 16)


def _seed_word(seed):
    z = (seed * 0x9E3779B97F4A7C15 + 0x632BE59BD9B4E019) & ((1 << 64) - 1)
    z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & ((1 << 64) - 1)
    return z ^ (z >> 31)


def _keys(layout, n, seed, absent=False):
    """n distinct uniformly random keys; those with absent=True never meet the others."""
    if layout == "packed32":
        start = (1 << 31) if absent else 0
        x = torch.arange(start, start + n + 8, dtype=torch.int64, device=_dev())
        k = _mix32(x ^ (_seed_word(seed) & 0x7FFFFFFF))
        k = k[k >= 2][:n]
        return torch.where(k >= 1 << 31, k - (1 << 32), k).to(torch.int32)
    start = (1 << 61) if absent else 0
    x = torch.arange(start, start + n, dtype=torch.int64, device=_dev())
    return _mix64(x ^ (_seed_word(seed) & ((1 << 60) - 1)))


def _gen(seed):
    g = torch.Generator(device=_dev())
    g.manual_seed(seed)
    return g


def _word(layout):
    return torch.int32 if layout == "packed32" else torch.int64


def _vals(layout, n, seed):
    return torch.randint(0, 1 << 30, (n,), generator=_gen(seed + 1), device=_dev()).to(_word(layout))


def _zipf(n, universe, s, seed):
    """Skewed keys: the inverse of the continuous power law x^-s on [1, universe + 1], floored, plus one."""
    u = torch.rand(n, generator=_gen(seed + 2), device=_dev(), dtype=torch.float64)
    top = float(universe + 1)
    if abs(s - 1.0) < 1e-9:
        x = torch.exp(u * math.log(top))
    else:
        x = (1.0 + u * (top ** (1.0 - s) - 1.0)) ** (1.0 / (1.0 - s))
    return x.floor().clamp(1, universe).to(torch.int64) + 1


def _cell(layout):
    return 8 if layout == "packed32" else 16


def _table(c, **kw):
    h = c.get("hash", "crc")
    t = lpht.Table(layout=lpht.PACKED32 if c["layout"] == "packed32" else lpht.KV64,
                   hash=lpht.HASH_MULSHIFT if h == "mul" else lpht.HASH_CRC32C_PAIR, mul=MUL if h == "mul" else 0, **kw)
    if c.get("tuned"):
        t.set_tuning(**TUNED)
    return t


def _arrays(c, seed):
    """The case's input arrays, made from the seed alone."""
    kind, layout = c["kind"], c.get("layout", "kv64")
    g = _gen(seed)
    if kind == "load_find":
        n = c["n"]
        keys, vals = _keys(layout, n, seed), _vals(layout, n, seed)
        order = torch.randperm(n, generator=g, device=_dev())
        return dict(keys=keys, vals=vals, hits=keys[order], want=vals[order], misses=_keys(layout, n, seed, True))
    if kind == "modify":
        n = c["n"]
        keys = _keys(layout, n + n // 2, seed)
        order = torch.randperm(n + n // 2, generator=g, device=_dev())
        return dict(keys=keys[:n].contiguous(), vals=_vals(layout, n, seed),
                    again=keys[n // 2:].contiguous(), again_vals=_vals(layout, n + n // 2 - n // 2, seed + 7),
                    added=keys[n // 4:n // 4 + n // 2].contiguous(), gone=keys[n // 3::2].contiguous(),
                    asked=keys[order].contiguous(), order=order)
    if kind == "lookup":
        st, n = c["stored"], c["n"]
        keys, vals = _keys(layout, st, seed), _vals(layout, st, seed)
        at = torch.randint(0, st, (n,), generator=g, device=_dev())
        absent = torch.rand(n, generator=g, device=_dev()) < 0.5
        asked = torch.where(absent, _keys(layout, n, seed, True), keys[at])
        return dict(keys=keys, vals=vals, asked=asked, want=torch.where(absent, torch.zeros_like(vals[at]), vals[at]),
                    present=(~absent).to(torch.uint8))
    if kind in ("count", "in_kernel"):
        n = c["n"]
        keys = _zipf(n, c["universe"], c["s"], seed)
        asked = torch.randperm(min(c["universe"], max(16, n // 8)), generator=g, device=_dev()) + 2
        return dict(keys=keys, asked=asked)
    if kind == "growing":
        n = c["n"]
        keys, vals = _keys(layout, n, seed), _vals(layout, n, seed)
        at = torch.randint(0, n, (max(1, n // 8),), generator=g, device=_dev())
        return dict(keys=keys, vals=vals, asked=keys[at], want=vals[at])
    if kind == "window":
        n = c["window"] + c["batch"] * c["steps"]
        keys = _keys(layout, n, seed)
        at = torch.randint(0, n, (max(1, n // 8),), generator=g, device=_dev())
        return dict(keys=keys, vals=_vals(layout, n, seed), asked=keys[at], at=at)
    if kind == "bulk":
        n, m = c["n"], c["m"]
        keys = _keys(layout, n + m // 2, seed)
        # a quarter of the build's keys come a second time; half of the merge's are in the table
        build = torch.cat([keys[:n - n // 4], keys[:n // 4]])[torch.randperm(n, generator=g, device=_dev())]
        merge = keys[n - n // 4 - (m - m // 2):][:m].contiguous()
        at = torch.randint(0, keys.numel(), (max(1, n // 4),), generator=g, device=_dev())
        return dict(build=build, vals=_vals(layout, n, seed), merge=merge, merge_vals=_vals(layout, m, seed + 7),
                    asked=keys[at])
    if kind == "strings":
        n = c["n"]
        lens = torch.randint(8, 41, (2 * n,), generator=g, device=_dev())
        offs = torch.zeros(2 * n + 1, dtype=torch.int64, device=_dev())
        offs[1:] = torch.cumsum(lens, 0)
        raw = torch.randint(0, 256, (int(offs[-1]),), generator=g, device=_dev(), dtype=torch.uint8)
        # every key distinct: its number in its first 8 bytes
        number = torch.arange(2 * n, dtype=torch.int64, device=_dev())
        for b in range(8):
            raw[offs[:-1] + b] = ((number >> (8 * b)) & 255).to(torch.uint8)
        return dict(bytes=raw, offs=offs[:n + 1].contiguous(), miss_offs=offs[n:].contiguous(),
                    vals=_vals("kv64", n, seed))
    raise ValueError(kind)


def _requests(c, seed):
    """Requests on random tables: lognormal sizes, Zipf keys, each key once in a request, 60/30/10 kinds."""
    shape, r = np.random.default_rng(17), np.random.default_rng(seed)
    caps = [int(e) for e in shape.integers(12, 21, size=c["tables"])]
    sizes = np.clip(np.rint(np.exp(shape.normal(math.log(c["median"]), 1.0, size=c["requests"]))), 64, 1 << 18).astype(int)
    tables = shape.integers(0, c["tables"], size=c["requests"])
    reqs = []
    for n, table in zip(sizes, tables):
        x = np.exp(r.random(4 * int(n) + 4000) * math.log(10.0 ** 8 + 1)).astype(np.uint64) + np.uint64(1)
        k = np.unique(x)
        r.shuffle(k)
        k = k[:n]
        reqs.append((int(table), k, r.choice(np.array([0, 1, 2], np.uint8), k.size, p=[0.6, 0.3, 0.1])))
    return caps, reqs


# ---------------------------------------------------------------- the pass

def prepare(case, seed):
    c = dict(case)
    if c["kind"] == "serving":
        caps, reqs = _requests(c, seed)
        srv = lpht.Server(caps, mode=lpht.SERVE_WAVES, max_inflight=64, streams=4)
        arr, outs, keep = srv.make_requests(reqs)
        return dict(c=c, srv=srv, arr=arr, vals=keep[2], flags=keep[3], keep=keep, outs=outs)
    s = dict(c=c, **_arrays(c, seed))
    if c["kind"] in ("load_find", "modify", "count"):
        s["table"] = _table(c, log2_capacity=c["log2_capacity"])
    elif c["kind"] == "lookup":
        s["table"] = _table(c, log2_capacity=c["log2_capacity"])
        s["table"].insert(s.pop("keys"), s.pop("vals"), flags=False)
    return s


def run(s):
    c = s["c"]
    return _RUN[c["kind"]](c, s)


def _run_load_find(c, s):
    t = s["table"]
    t.clear()
    flags = t.insert(s["keys"], s["vals"], flags=c["flags"])
    out = dict(hit=t.find(s["hits"]), miss=t.find(s["misses"]))
    if c["flags"]:
        out["inserted"] = flags
    return out


def _run_modify(c, s):
    t = s["table"]
    t.clear()
    out = dict(inserted=t.insert(s["keys"], s["vals"]))
    out["upserted"] = t.insert_or_update(s["again"], s["again_vals"], op=lpht.ASSIGN)
    out["updated"] = t.update(s["added"], op=lpht.ADD)
    out["erased"] = t.erase(s["gone"])
    out["found"] = t.find(s["asked"])
    return out


def _run_lookup(c, s):
    return s["table"].find(s["asked"])


def _run_count(c, s):
    t = s["table"]
    t.clear()
    t.insert_or_update(s["keys"], op=lpht.ADD, flags=False)
    return t.find(s["asked"])


def _run_growing(c, s):
    t = _table(c, log2_capacity=12, auto_grow=True)
    b, n = c["batch"], c["n"]
    flags = [t.insert(s["keys"][lo:lo + b], s["vals"][lo:lo + b]) for lo in range(0, n, b)]
    found = t.find(s["asked"])
    used, live = t.count()
    t.close()
    return dict(inserted=flags, found=found, live=live)


def _run_in_kernel(c, s):
    t = _table(c, log2_capacity=12, auto_grow=True)
    t.insert_async(s["keys"], add=True, flags=False)
    found = t.find(s["asked"])
    used, live = t.count()
    t.close()
    return dict(found=found, live=live)


def _run_window(c, s):
    t = _table(c, log2_capacity=c["log2_capacity"], auto_grow=True)
    w, b = c["window"], c["batch"]
    k, v = s["keys"], s["vals"]
    t.insert(k[:w], v[:w], flags=False)
    inserted, erased = [], []
    for lo in range(0, b * c["steps"], b):
        inserted.append(t.insert(k[w + lo:w + lo + b], v[w + lo:w + lo + b]))
        erased.append(t.erase(k[lo:lo + b]))
    found = t.find(s["asked"])
    used, live = t.count()
    t.close()
    return dict(inserted=inserted, erased=erased, found=found, live=live)


def _run_bulk(c, s):
    t = _table(c, log2_capacity=c["log2_capacity"])
    t.build(s["build"], s["vals"], op=lpht.ADD)
    t.merge(s["merge"], s["merge_vals"], op=lpht.ASSIGN)
    found = t.find(s["asked"])
    used, live = t.count()
    t.close()
    return dict(found=found, live=live)


def _run_strings(c, s):
    n = c["n"]
    L = lpht._str_lib()  # the C ABI, as a program with its keys already on the GPU calls it
    t = lpht.StrTable(log2_capacity=c["log2_capacity"], pool_bytes=s["bytes"].numel() // 2 + 20 * n + 4096)
    p = lpht._ptr
    stream = lpht._stream_handle(None)
    flags, hit, miss = (torch.empty(n, dtype=torch.uint8, device=_dev()) for _ in range(3))
    got, none = (torch.empty(n, dtype=torch.int64, device=_dev()) for _ in range(2))
    for rc in (L.lpht_str_insert(t._h, p(s["bytes"]), p(s["offs"]), n, p(s["vals"]), p(flags), stream),
               L.lpht_str_find(t._h, p(s["bytes"]), p(s["offs"]), n, p(got), p(hit), stream),
               L.lpht_str_find(t._h, p(s["bytes"]), p(s["miss_offs"]), n, p(none), p(miss), stream)):
        if rc != lpht.OK:
            raise lpht.LphtError(rc, "string keys")
    t.close()
    return dict(inserted=flags, hit=(got, hit), miss=(none, miss))


def _run_serving(c, s):
    s["srv"].run_closed_loop(s["arr"], c["clients"])
    return dict(vals=s["vals"], flags=s["flags"])


_RUN = dict(load_find=_run_load_find, modify=_run_modify, lookup=_run_lookup, count=_run_count,
            growing=_run_growing, in_kernel=_run_in_kernel, window=_run_window, bulk=_run_bulk,
            strings=_run_strings, serving=_run_serving)


# ---------------------------------------------------------------- what a pass cannot do without

def work(case):
    """Bytes of the inputs, outputs and cells that a pass must read or write once; the table does no arithmetic to speak of
    (one operation per table operation stands for the hash)."""
    c = case
    kind = c["kind"]
    cell = _cell(c.get("layout", "kv64"))
    kb = cell // 2
    n = c.get("n", 0)
    cells = cell << c.get("log2_capacity", 0)
    if kind == "load_find":
        # the table cleared, n cells filled, 2n cells looked at
        b, ops = cells + n * (2 * kb + cell + c["flags"]) + 2 * n * (kb + cell + kb + 1), 3 * n
    elif kind == "modify":
        a = n + n // 2
        b = cells + n * (2 * kb + cell + 1) + n * (2 * kb + cell + 1) + (n // 2) * (kb + 2 * cell + 1)
        b += (a // 2) * (kb + 2 * cell + 1) + a * (kb + cell + kb + 1)
        ops = 4 * n
    elif kind == "lookup":
        b, ops = n * (kb + cell + kb + 1), n
    elif kind == "count":
        d = _distinct(n, c["universe"], c["s"])
        q = max(16, n // 8)
        b, ops = cells + n * kb + d * cell + q * (2 * kb + cell + 1), n + q
    elif kind == "growing":
        # every key written once, and the final table written once
        fin = cell << max(12, math.ceil(math.log2(2 * n)))
        b, ops = fin + n * (2 * kb + 1) + (n // 8) * (2 * kb + cell + 1), n + n // 8
    elif kind == "in_kernel":
        d = _distinct(n, c["universe"], c["s"])
        fin = cell << max(12, math.ceil(math.log2(2 * d)))
        b, ops = fin + n * kb + (n // 8) * (2 * kb + cell + 1), n + n // 8
    elif kind == "window":
        m = c["window"] + c["batch"] * c["steps"]
        b = cells + m * (2 * kb + cell) + c["batch"] * c["steps"] * (kb + cell + 2) + (m // 8) * (2 * kb + cell + 1)
        ops = m + c["batch"] * c["steps"] + m // 8
    elif kind == "bulk":
        # the batch read, the table written; then the table read and written again with the merge
        b = n * 2 * kb + cells + c["m"] * 2 * kb + 2 * cells + (n // 4) * (2 * kb + cell + 1)
        ops = n + c["m"] + n // 4
    elif kind == "strings":
        # 24 key bytes and an 8-byte offset each; pool record and cell written, then read
        b, ops = 16 * (1 << c["log2_capacity"]) + n * (24 + 8 + 8 + 28 + 16 + 1) + 2 * n * (24 + 8 + 16 + 9) + n * 28, 3 * n
    else:
        m = c["requests"] * c["median"] * math.exp(0.5)
        b, ops = m * (8 + 1 + 8 + 1 + 16), m
    return dict(bytes=float(b), flops=float(ops))


def _distinct(n, universe, s):
    """Expected distinct keys of n draws of the power law (in steps over the logarithm of the rank)."""
    e = np.linspace(0.0, math.log(universe + 1.0), 4001)
    lo, hi = np.exp(e[:-1]), np.exp(e[1:])
    if abs(s - 1.0) < 1e-9:
        mass = (e[1:] - e[:-1]) / math.log(universe + 1.0)
    else:
        mass = (hi ** (1 - s) - lo ** (1 - s)) / ((universe + 1.0) ** (1 - s) - 1.0)
    ranks = np.maximum(1.0, hi - lo)
    return float(np.sum(np.minimum(hi - lo, ranks) * -np.expm1(-n * mass / ranks)))


# ---------------------------------------------------------------- results by sorting and indexing

def _look_up(keys, vals, asked):
    """(values, found) of `asked` in the distinct keys `keys`."""
    order = torch.argsort(keys)
    k = keys[order]
    at = torch.searchsorted(k, asked).clamp(max=k.numel() - 1)
    hit = k[at] == asked
    v = vals[order][at]
    return torch.where(hit, v, torch.zeros_like(v)), hit.to(torch.uint8)


def exact(case, seed):
    c = dict(case)
    kind = c["kind"]
    if kind == "serving":
        return None
    a = _arrays(c, seed)
    one = lambda m: torch.ones(m, dtype=torch.uint8, device=_dev())  # noqa: E731
    if kind == "load_find":
        n = c["n"]
        zero = torch.zeros(n, dtype=torch.uint8, device=_dev())
        out = dict(hit=(a["want"], one(n)), miss=(torch.zeros_like(a["vals"]), zero))
        if c["flags"]:
            out["inserted"] = one(n)
        return out
    if kind == "modify":
        n = c["n"]
        m = n + n // 2
        at = torch.arange(m, device=_dev())
        val = torch.zeros(m, dtype=a["vals"].dtype, device=_dev())
        val[:n] = a["vals"]
        val[n // 2:] = a["again_vals"]
        val[n // 4:n // 4 + n // 2] += 1
        live = torch.ones(m, dtype=torch.bool, device=_dev())
        live[n // 3::2] = False
        val = torch.where(live, val, torch.zeros_like(val))
        return dict(inserted=one(n), upserted=(at[n // 2:] >= n).to(torch.uint8), updated=one(n // 2),
                    erased=one(a["gone"].numel()), found=(val[a["order"]], live[a["order"]].to(torch.uint8)))
    if kind == "lookup":
        return a["want"], a["present"]
    if kind in ("count", "in_kernel"):
        k, v = torch.unique(a["keys"], return_counts=True)
        found = _look_up(k, v, a["asked"])
        return found if kind == "count" else dict(found=found, live=k.numel())
    if kind == "growing":
        n, b = c["n"], c["batch"]
        return dict(inserted=[one(min(b, n - lo)) for lo in range(0, n, b)],
                    found=(a["want"], one(a["want"].numel())), live=n)
    if kind == "window":
        b, st = c["batch"], c["steps"]
        at = a["at"]
        present = at >= b * st
        v = a["vals"][at]
        return dict(inserted=[one(b) for _ in range(st)], erased=[one(b) for _ in range(st)],
                    found=(torch.where(present, v, torch.zeros_like(v)), present.to(torch.uint8)), live=c["window"])
    if kind == "bulk":
        k, where = torch.unique(a["build"], return_inverse=True)
        v = torch.zeros_like(k).index_add_(0, where, a["vals"])
        new = ~torch.isin(k, a["merge"])
        k, v = torch.cat([k[new], a["merge"]]), torch.cat([v[new], a["merge_vals"]])
        return dict(found=_look_up(k, v, a["asked"]), live=k.numel())
    n = c["n"]
    zero = torch.zeros(n, dtype=torch.uint8, device=_dev())
    return dict(inserted=one(n), hit=(a["vals"], one(n)), miss=(torch.zeros_like(a["vals"]), zero))
