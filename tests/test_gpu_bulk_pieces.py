"""Grouped calls that run in pieces: two and three ragged pieces with keys in several of
them, and groups whose tables share a run, fill one, span several or get too few
operations, against the oracle (the instrumented library's pieces hold 2^18 operations);
one call beyond the product library's 2^27; and the wide split of calls from 2^22 on."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2509_16407_amd as hw
from paper_2509_16407_amd import workloads as w
from gpu_util import busy_lock_queues, dev, host, per_key_counts, u8

pytestmark = pytest.mark.gpu

PIECE = 1 << 18


def dump_equal(t, om):
    gk, gv = (host(x, t.kv_bits) for x in t.export())
    o = np.argsort(gk)
    ok, ov = om.dump()
    assert np.array_equal(gk[o], ok) and np.array_equal(gv[o], ov)
    assert busy_lock_queues(t) == 0


def run_and_check(t, om, seed, n, combine=("sum", oracle.SUM)):
    """SUM upserts of n operations on 0.8 n keys, all over the call, then erases of half of
    it and of absent keys."""
    bits = t.kv_bits
    pool = w.distinct_keys(seed, int(0.8 * n) + 4000, key_bits=bits)
    u = int(0.8 * n)
    k = pool[w.uniform_below(seed + 1, 0, n, u)]
    k[::50021] = np.uint64((1 << bits) - 1)
    v = w.splitmix64(seed + 2, 0, n) & np.uint64(0xFFFFF)
    if not t.design.startswith("P2"):
        assert t._scratch(hw.OPS["upsert"], n, 0, None) is not None
    st, ost = u8(t.upsert(dev(k, bits), dev(v, bits))), om.upsert(k, v)
    for c in (hw.ST_DONE, hw.ST_EXISTED, hw.ST_INVALID):
        assert per_key_counts(k, st, c) == per_key_counts(k, ost, c), c
    dump_equal(t, om)
    e = np.concatenate([k[: n - 4000], pool[u:]])
    e[1::2] = pool[:u][w.uniform_below(seed + 3, 0, len(e) // 2, u // 2)]
    assert t._scratch(hw.OPS["erase"], n, 0, None) is not None
    st, ost = u8(t.erase(dev(e, bits))), om.erase(e)
    for c in (hw.ST_DONE, hw.ST_MISS, hw.ST_INVALID):
        assert per_key_counts(e, st, c) == per_key_counts(e, ost, c), c
    dump_equal(t, om)


@pytest.mark.parametrize("design,bits,bucket,tile", [("DOUBLE_M", 64, 32, 4), ("DOUBLE", 32, 16, 4), ("ICEBERG", 64, 32, 8),
                                                     ("P2_M", 64, 32, 4)])
@pytest.mark.parametrize("n", [PIECE + 1, 2 * PIECE + 77777])
def test_pieces_against_oracle(design, bits, bucket, tile, n):
    t = hw.Table(1 << (19 if n < 2 * PIECE else 20), design, kv_bits=bits, bucket=bucket, tile=tile, instrumented=True)
    run_and_check(t, oracle.OracleMap(key_bits=bits), w.stream_seed(300 + hw.DESIGNS[design], n), n)


@pytest.mark.parametrize("design,bits,bucket,tile", [("DOUBLE_M", 64, 32, 4), ("P2_M", 64, 32, 4), ("DOUBLE", 32, 16, 4)])
def test_wide_split_against_oracle(design, bits, bucket, tile):
    t = hw.Table(1 << 23, design, kv_bits=bits, bucket=bucket, tile=tile)
    run_and_check(t, oracle.OracleMap(key_bits=bits), w.stream_seed(310 + hw.DESIGNS[design], bits), (1 << 22) + 12345)


@pytest.mark.parametrize("design,bits,bucket,tile", [("DOUBLE", 32, 16, 4), ("ICEBERG_M", 64, 32, 4)])
def test_group_in_runs_against_oracle(design, bits, bucket, tile, monkeypatch):
    """Tables of 100 to 600,001 operations: runs of many tables, of one, of a piece of one;
    a run of tables that all get too few operations; an empty table at each end."""
    instr = hw.lib(instrumented=True)
    monkeypatch.setattr(hw, "lib", lambda instrumented=False: instr)
    ns = [0, 100, 9000, 70000, 200000, 600001, 3000, 3000, 250000, PIECE, 5, 131000, 0]
    caps = [1 << 10, 1 << 10, 1 << 13, 1 << 16, 1 << 18, 1 << 19, 1 << 18, 1 << 18, 1 << 23, 1 << 18, 1 << 10, 1 << 17, 1 << 10]
    tables = [hw.Table(c, design, kv_bits=bits, bucket=bucket, tile=tile, instrumented=True) for c in caps]
    m = hw.Multi(tables)
    ks, vs = [], []
    for i, (n, c) in enumerate(zip(ns, caps)):
        seed = w.stream_seed(320 + i, bits)
        pool = w.distinct_keys(seed, max(1, int(0.6 * min(c, n or 1))), key_bits=bits)
        ks.append(pool[w.uniform_below(seed + 1, 0, n, len(pool))] if n else np.empty(0, np.uint64))
        vs.append(w.splitmix64(seed + 2, 0, n) & np.uint64(0xFFFFF))
    offs = [0] + np.cumsum(ns).tolist()
    keys, vals = np.concatenate(ks), np.concatenate(vs)
    arr = (ctypes.c_uint64 * len(offs))(*offs)
    need = m._scratch(arr, len(keys), 0, None)
    # bounded by a run's operations, not by the call's
    assert need is not None and need.numel() < 100 * PIECE < 100 * len(keys)
    oms = [oracle.OracleMap(key_bits=bits) for _ in ns]
    for _ in range(2):
        st = u8(m.upsert(offs, dev(keys, bits), dev(vals, bits)))
        for i, k in enumerate(ks):
            if len(k):
                ost = oms[i].upsert(k, vs[i])
                for c in (hw.ST_DONE, hw.ST_EXISTED):
                    assert per_key_counts(k, st[offs[i]: offs[i + 1]], c) == per_key_counts(k, ost, c), (i, c)
    for t, om in zip(tables, oms):
        dump_equal(t, om)


MIX32 = [("DOUBLE", 16, 4), ("DOUBLE", 16, 8), ("DOUBLE", 64, 32)]
MIX64 = [("DOUBLE_M", 32, 4), ("ICEBERG_M", 32, 4), ("CHAINING", 0, 0)]


@pytest.mark.parametrize("bits,mix,grouped", [(32, MIX32, True), (64, MIX64, True), (64, [("P2_M", 32, 4)] + MIX64[1:], False)])
def test_group_of_several_configurations_against_oracle(bits, mix, grouped):
    """Tables of three configurations in turn, the first configuration with most of the
    operations, the third with a table of a few; another one's tables get none.  Grouped from
    2^20 operations per configuration on, where each configuration has a grouped upsert."""
    cap = 1 << 20
    each = 5 * cap // 8
    ns = [each, 60000, 900, each, 0, 70000, each, 3, 0, each, 7, 0, 3 * cap - 4 * each - 130910]
    tables = [hw.Table(cap if n > 60000 else 1 << 17, d, kv_bits=bits, bucket=b, tile=t)
              for n, (d, b, t) in zip(ns, mix * 5)]
    tables.append(hw.Table(1 << 10, "DOUBLE", kv_bits=bits, bucket=16, tile=8 if bits == 64 else 4))
    ns.append(0)
    m = hw.Multi(tables)
    assert m.kernel()[0] != "solo" and sum(ns) == 3 * cap
    ks, vs = [], []
    for i, n in enumerate(ns):
        seed = w.stream_seed(340 + i, bits)
        pool = w.distinct_keys(seed, max(1, int(0.6 * n)), key_bits=bits)
        ks.append(pool[w.uniform_below(seed + 1, 0, n, len(pool))] if n else np.empty(0, np.uint64))
        vs.append(w.splitmix64(seed + 2, 0, n) & np.uint64(0xFFFFF))
    offs = [0] + np.cumsum(ns).tolist()
    keys, vals = np.concatenate(ks), np.concatenate(vs)
    arr = (ctypes.c_uint64 * len(offs))(*offs)
    assert (m._scratch(arr, len(keys), 0, None) is not None) == grouped
    fewer = (ctypes.c_uint64 * len(offs))(0, *[x - 1 for x in offs[1:]])
    assert m._scratch(fewer, len(keys) - 1, 0, None) is None
    oms = [oracle.OracleMap(key_bits=bits) for _ in ns]
    for _ in range(2):
        st = u8(m.upsert(offs, dev(keys, bits), dev(vals, bits)))
        for i, k in enumerate(ks):
            if len(k):
                ost = oms[i].upsert(k, vs[i])
                for c in (hw.ST_DONE, hw.ST_EXISTED):
                    assert per_key_counts(k, st[offs[i]: offs[i + 1]], c) == per_key_counts(k, ost, c), (i, c)
    for t, om in zip(tables, oms):
        dump_equal(t, om)


def test_a_call_beyond_one_piece():
    """2^27 and 12,345 more operations on 10^8 keys, against sums worked out with torch:
    key i appears once, or twice if i < n - 10^8."""
    n, u = (1 << 27) + 12345, 100_000_000
    t = hw.Table(1 << 27, "DOUBLE_M")
    z = torch.arange(1, u + 1, dtype=torch.int64, device="cuda") * -7046029254386353131
    z = (z ^ ((z >> 29) & ((1 << 35) - 1))) * -4658895280553007687
    z &= (1 << 63) - 1
    z = torch.unique(z)
    u = z.numel()
    k = torch.cat([z, z[: n - u]])
    v = torch.arange(n, dtype=torch.int64, device="cuda")
    assert t._scratch(hw.OPS["upsert"], n, 0, None) is not None
    st = t.upsert(k, v)
    first = st == hw.ST_DONE
    assert int(first.sum()) == u and int((st == hw.ST_EXISTED).sum()) == n - u
    assert bool((first[: n - u] ^ first[u:]).all()) and bool(first[n - u: u].all())
    f, x = t.query(z)
    want = torch.arange(u, dtype=torch.int64, device="cuda")
    want[: n - u] += torch.arange(u, n, dtype=torch.int64, device="cuda")
    assert bool((f == hw.ST_DONE).all()) and bool((x == want).all())
    e = t.erase(k) == hw.ST_DONE
    assert int(e.sum()) == u and bool((e[: n - u] ^ e[u:]).all()) and t.size() == 0
