"""Upserts over a group of tables, grouped by bucket in launches over all tables: every
table against the oracle, with capacities on both sides of one and two split
levels, tables that get no or too few operations, duplicates, reserved keys and
skew beyond a bin's room; and the groups that keep the plain launch."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2509_16407_amd as hw
from paper_2509_16407_amd import workloads as w
from gpu_util import busy_lock_queues, dev, host, per_key_counts, u8

pytestmark = pytest.mark.gpu

CASES = [("DOUBLE", 32, 16, 4), ("DOUBLE_M", 32, 32, 4), ("DOUBLE", 64, 8, 8), ("DOUBLE_M", 64, 32, 4),
         ("ICEBERG", 64, 32, 8), ("ICEBERG_M", 64, 32, 4), ("CHAINING", 64, 7, 8)]
COMB = {"sum": oracle.SUM, "keep": oracle.KEEP, "replace": oracle.REPLACE, "min": oracle.MIN, "max": oracle.MAX}
# (capacity, operations per slot): one part, several, two levels; few operations; none
SHAPES = [(1 << 10, 1.7), (1 << 13, 0.9), (1 << 12, 0.01), (1 << 10, 0.0), (1 << 20, 1.7), (1 << 16, 1.2), (1 << 10, 3.0)]


def scratch_of(m, offs, n, combine="sum"):
    return m._scratch((ctypes.c_uint64 * len(offs))(*offs), n, hw.COMBINES[combine], None)


def batches(seed, bits, combine):
    top = np.uint64((1 << bits) - 1)
    for i, (cap, per) in enumerate(SHAPES):
        n = int(cap * per) + (1 if per else 0)
        u = max(1, min(int(0.6 * cap), n))
        pool = w.distinct_keys(seed + i, u, key_bits=bits)
        k = pool[w.uniform_below(seed + 100 + i, 0, n, u)] if n else np.empty(0, np.uint64)
        if i == 6:
            k[: n // 2] = pool[3]  # more than a bin's room
        if i == 4:
            k[::100003] = top
        v = w.value_of(k, bits) if combine in ("keep", "replace") else w.splitmix64(seed + 200 + i, 0, n) & np.uint64(0xFFFFFF)
        yield cap, k, v


@pytest.mark.parametrize("design,bits,bucket,tile", CASES, ids=["%s-u%d" % c[:2] for c in CASES])
@pytest.mark.parametrize("combine", list(COMB))
def test_group_upsert_against_oracle(design, bits, bucket, tile, combine):
    b = list(batches(w.stream_seed(250 + hw.DESIGNS[design], bits), bits, combine))
    tables = [hw.Table(cap, design, kv_bits=bits, bucket=bucket, tile=tile) for cap, _, _ in b]
    m = hw.Multi(tables)
    offs = [0] + np.cumsum([len(k) for _, k, _ in b]).tolist()
    keys, vals = np.concatenate([k for _, k, _ in b]), np.concatenate([v for _, _, v in b])
    assert scratch_of(m, offs, len(keys), combine) is not None
    oms = [oracle.OracleMap(key_bits=bits) for _ in b]
    for _ in range(2):  # absent keys, then present ones
        st = u8(m.upsert(offs, dev(keys, bits), dev(vals, bits), combine=combine))
        for i, (_, k, v) in enumerate(b):
            if len(k) == 0:
                continue
            ost = oms[i].upsert(k, v, combine=COMB[combine])
            for code in (hw.ST_DONE, hw.ST_EXISTED, hw.ST_INVALID):
                assert per_key_counts(k, st[offs[i]: offs[i + 1]], code) == per_key_counts(k, ost, code), (i, code)
    for t, om in zip(tables, oms):
        gk, gv = (host(x, bits) for x in t.export())
        o = np.argsort(gk)
        ok, ov = om.dump()
        assert np.array_equal(gk[o], ok) and np.array_equal(gv[o], ov)
        assert busy_lock_queues(t) == 0


def test_groups_that_keep_the_plain_launch():
    """Two configurations, two-choice tables, few operations, most of them in tables with
    too few, merging tables, and a call under capture."""
    offs, n = [0, 100000, 200000], 200000
    mk = lambda *a, **k: hw.Table(1 << 17, *a, **k)
    assert scratch_of(hw.Multi([mk("DOUBLE"), mk("DOUBLE")]), offs, n) is not None
    assert scratch_of(hw.Multi([mk("DOUBLE"), mk("DOUBLE_M")]), offs, n) is None
    assert scratch_of(hw.Multi([mk("P2_M"), mk("P2_M")]), offs, n) is None
    small = hw.Multi([hw.Table(1 << 10, "DOUBLE"), hw.Table(1 << 10, "DOUBLE")])
    assert scratch_of(small, [0, 1000, 2047], 2047) is None and scratch_of(small, [0, 1000, 2048], 2048) is not None
    assert scratch_of(hw.Multi([hw.Table(1 << 20, "DOUBLE"), mk("DOUBLE")]), [0, 150000, 200000], n) is None
    agg = hw.Multi([mk("DOUBLE", flags=hw.F_AGGREGATE), mk("DOUBLE")])
    assert scratch_of(agg, offs, n) is None and scratch_of(agg, offs, n, "replace") is not None


@pytest.mark.parametrize("null_status", [False, True])
def test_group_upsert_without_scratch_or_status(null_status):
    """The C-ABI call with too little scratch memory is the plain call; no status array."""
    k = w.distinct_keys(w.stream_seed(260, 1), 100000)
    dk, dv = dev(k), dev(w.value_of(k))
    tables = [hw.Table(1 << 17, "DOUBLE_M"), hw.Table(1 << 16, "DOUBLE_M")]
    m = hw.Multi(tables)
    offs = (ctypes.c_uint64 * 3)(0, 60000, 100000)
    sc = m._scratch(offs, 100000, 0, None)
    L, s = hw.lib(), hw._stream(None)
    st = torch.empty(100000, dtype=torch.uint8, device="cuda")
    p = None if null_status else hw._ptr(st)
    o = ctypes.cast(offs, ctypes.c_void_p)
    for size in (sc.numel(), sc.numel() - 1):
        assert L.hwave_multi_upsert_scratch(m.h, o, hw._ptr(dk), hw._ptr(dv), 0, p, hw._ptr(sc), size, s) == 0
    for t, a, b in ((tables[0], 0, 60000), (tables[1], 60000, 100000)):
        f, v = t.query(dk[a:b])
        assert bool((f == hw.ST_DONE).all()) and np.array_equal(host(v), w.value_of(k[a:b]) * np.uint64(2))
        assert t.size() == b - a
    if not null_status:
        assert bool((st == hw.ST_EXISTED).all())
