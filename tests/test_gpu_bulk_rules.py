"""Which calls are grouped by bucket: the smallest share of a table's slots per design,
bucket and kind of call; tables that never erase keep the plain call where few
operations share a key."""
import ctypes

import numpy as np
import pytest

import paper_2509_16407_amd as hw
from paper_2509_16407_amd import workloads as w
from gpu_util import dev, host, u8

pytestmark = pytest.mark.gpu

# design, key bits, bucket, tile, kind, capacity, operations per slot below the line and above it
LINES = [("DOUBLE", 64, 8, 8, "insert", 1 << 16, 0.27, 0.30), ("DOUBLE", 64, 8, 8, "upsert", 1 << 15, 0.27, 0.30),
         ("DOUBLE", 64, 8, 8, "erase", 1 << 14, 0.30, 0.33), ("DOUBLE", 32, 8, 4, "insert", 1 << 15, 0.19, 0.22),
         ("DOUBLE", 32, 16, 4, "insert", 1 << 15, 0.15, 0.17), ("DOUBLE_M", 64, 16, 4, "upsert", 1 << 16, 0.12, 0.14),
         ("DOUBLE_M", 64, 32, 4, "upsert", 1 << 16, 0.09, 0.11), ("P2_M", 64, 16, 4, "erase", 1 << 15, 0.12, 0.14),
         ("P2_M", 64, 32, 4, "erase", 1 << 15, 0.09, 0.11), ("ICEBERG", 64, 32, 8, "insert", 1 << 17, 0.08, 0.11),
         ("P2", 64, 32, 8, "erase", 1 << 16, 0.23, 0.26), ("DOUBLE", 64, 16, 8, "erase", 1 << 16, 0.23, 0.26),
         ("ICEBERG", 64, 32, 8, "upsert", 1 << 17, 0.08, 0.11), ("ICEBERG_M", 64, 32, 4, "insert", 1 << 17, 0.07, 0.09),
         ("ICEBERG_M", 32, 32, 4, "upsert", 1 << 17, 0.07, 0.09), ("CHAINING", 64, 0, 0, "erase", 1 << 15, 0.33, 0.39),
         ("CHAINING", 64, 0, 0, "upsert", 1 << 15, 0.65, 0.71),
         # from 2^23 buckets on
         ("DOUBLE_M", 64, 32, 4, "insert", 1 << 28, 0.19, 0.21), ("DOUBLE_M", 64, 16, 4, "upsert", 1 << 27, 0.19, 0.21),
         ("DOUBLE_M", 64, 32, 4, "upsert", 1 << 27, 0.09, 0.11), ("DOUBLE_M", 64, 32, 4, "erase", 1 << 28, 0.09, 0.11),
         ("DOUBLE_M", 64, 32, 8, "insert", 1 << 28, 0.09, 0.11), ("DOUBLE_M", 32, 32, 4, "insert", 1 << 28, 0.09, 0.11)]


@pytest.mark.parametrize("design,bits,bucket,tile,kind,cap,below,above", LINES, ids=["%s-u%d-b%d-t%d-%s-%d" % c[:6] for c in LINES])
def test_least_share_of_the_slots(design, bits, bucket, tile, kind, cap, below, above):
    t = hw.Table(cap, design, kv_bits=bits, bucket=bucket, tile=tile)
    grouped = lambda per: t._scratch(hw.OPS[kind], int(per * cap), hw.COMBINES["keep" if kind == "insert" else "sum"], None) is not None
    assert not grouped(below) and grouped(above)


@pytest.mark.parametrize("design", ["DOUBLE", "DOUBLE_M", "ICEBERG", "ICEBERG_M", "CHAINING"])
def test_tables_that_never_erase_keep_the_plain_call(design):
    """Their plain upserts of present keys take no lock."""
    cap, n = 1 << 16, 60000
    mk = lambda flags: [hw.Table(cap, design, flags=flags) for _ in range(2)]
    for flags in (0, hw.F_NO_ERASE):
        ts = mk(flags)
        for op, c in (("insert", 1), ("upsert", 0), ("upsert", 2)):
            assert (ts[0]._scratch(hw.OPS[op], n, c, None) is not None) == (flags == 0)
        m = hw.Multi(ts)
        assert (m._scratch((ctypes.c_uint64 * 3)(0, n, 2 * n), 2 * n, 0, None) is not None) == (flags == 0)


def test_large_calls_on_tables_that_never_erase():
    """From one operation per slot on: in groups of 2^17 operations, and alone in 2^24 slots."""
    def alone(design, cap, n):
        return hw.Table(cap, design, flags=hw.F_NO_ERASE)._scratch(hw.OPS["upsert"], n, 0, None) is not None

    def group(design, tables, n):
        m = hw.Multi([hw.Table(1 << 13, design, flags=hw.F_NO_ERASE) for _ in range(tables)])
        return m._scratch((ctypes.c_uint64 * (tables + 1))(*[n * i for i in range(tables + 1)]), n * tables, 0, None) is not None
    assert alone("DOUBLE_M", 1 << 24, 1 << 24) and not alone("DOUBLE_M", 1 << 24, (1 << 24) - 1)
    assert not alone("DOUBLE_M", 1 << 23, 1 << 24) and not alone("CHAINING", 1 << 24, 1 << 25) and not alone("ICEBERG", 1 << 24, 1 << 25)
    assert group("DOUBLE", 16, 1 << 13) and not group("DOUBLE", 15, 1 << 13) and not group("DOUBLE", 20, 8000)
    assert group("CHAINING", 20, 12000) and not group("ICEBERG_M", 20, 12000)


@pytest.mark.parametrize("design", ["DOUBLE", "DOUBLE_M", "CHAINING"])
def test_group_of_tables_that_never_erase(design):
    """Grouped SUM upserts, fresh and of present keys, beside a table with too few operations."""
    n, u, tables = 20000, 9000, 8
    ts = [hw.Table(1 << 14, design, flags=hw.F_NO_ERASE) for _ in range(tables)]
    m = hw.Multi(ts)
    pool = w.distinct_keys(w.stream_seed(330, hw.DESIGNS[design]), u * tables).reshape(tables, u)
    pick = w.uniform_below(331, 0, n * tables, u).reshape(tables, n)
    ns = [n] * (tables - 1) + [5000]
    keys = np.concatenate([pool[i][pick[i][:c]] for i, c in enumerate(ns)])
    offs = [0] + np.cumsum(ns).tolist()
    assert m._scratch((ctypes.c_uint64 * len(offs))(*offs), len(keys), 0, None) is not None
    for times in (1, 2):
        st = u8(m.upsert(offs, dev(keys), dev(np.ones(len(keys), np.uint64))))
        for i, t in enumerate(ts):
            k, c = np.unique(keys[offs[i]: offs[i + 1]], return_counts=True)
            assert (st[offs[i]: offs[i + 1]] == hw.ST_DONE).sum() == (len(k) if times == 1 else 0)
            f, v = t.query(dev(k))
            assert bool((f == hw.ST_DONE).all()) and np.array_equal(host(v), c.astype(np.uint64) * np.uint64(times))
            assert t.size() == len(k)


@pytest.mark.parametrize("design,least_us", [("DOUBLE", 1000), ("P2_M", 1000), ("CHAINING", 1000), ("ICEBERG", 4000), ("ICEBERG_M", 4000)])
def test_tables_with_little_patience_keep_the_plain_calls(design, least_us):
    """Their writers would time out beside a block that holds a bucket's lock for a part."""
    cap, n = 1 << 16, 60000
    for us in (0, least_us, least_us - 1, 10):
        ts = [hw.Table(cap, design, lock_timeout_us=us) for _ in range(2)]
        patient = us in (0, least_us)
        assert (ts[0]._scratch(hw.OPS["erase"], n, 0, None) is not None) == patient
        if design != "P2_M":
            assert (ts[0]._scratch(hw.OPS["upsert"], n, 0, None) is not None) == patient
            m = hw.Multi(ts)
            assert (m._scratch((ctypes.c_uint64 * 3)(0, n, 2 * n), 2 * n, 0, None) is not None) == patient


def test_groups_of_tables_with_few_operations_each():
    """A block per table pays from 64 operations on."""
    m = hw.Multi([hw.Table(1 << 8, "DOUBLE_M") for _ in range(100)])
    grouped = lambda n: m._scratch((ctypes.c_uint64 * 101)(*[n * i for i in range(101)]), 100 * n, 0, None) is not None
    assert grouped(64) and not grouped(63)
