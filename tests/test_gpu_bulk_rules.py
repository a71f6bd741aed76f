"""Which calls are grouped by bucket: the smallest share of a table's slots per design,
bucket and kind of call; tables that never erase keep the plain call."""
import ctypes

import pytest

import paper_2509_16407_amd as hw

pytestmark = pytest.mark.gpu

# design, key bits, bucket, tile, kind, capacity, operations per slot below the line and above it
LINES = [("DOUBLE", 64, 8, 8, "insert", 1 << 16, 0.27, 0.30), ("DOUBLE", 64, 8, 8, "upsert", 1 << 15, 0.27, 0.30),
         ("DOUBLE", 64, 8, 8, "erase", 1 << 14, 0.30, 0.33), ("DOUBLE", 32, 8, 4, "insert", 1 << 15, 0.19, 0.22),
         ("DOUBLE", 32, 16, 4, "insert", 1 << 15, 0.15, 0.17), ("DOUBLE_M", 64, 16, 4, "upsert", 1 << 16, 0.12, 0.14),
         ("DOUBLE_M", 64, 32, 4, "upsert", 1 << 16, 0.09, 0.11), ("P2_M", 64, 16, 4, "erase", 1 << 15, 0.12, 0.14),
         ("P2_M", 64, 32, 4, "erase", 1 << 15, 0.09, 0.11), ("ICEBERG", 64, 32, 8, "insert", 1 << 17, 0.13, 0.16),
         ("ICEBERG", 64, 32, 8, "upsert", 1 << 17, 0.08, 0.11), ("ICEBERG_M", 64, 32, 4, "insert", 1 << 17, 0.11, 0.13),
         ("ICEBERG_M", 32, 32, 4, "insert", 1 << 17, 0.11, 0.13), ("CHAINING", 64, 0, 0, "erase", 1 << 15, 0.33, 0.39),
         ("CHAINING", 64, 0, 0, "upsert", 1 << 15, 0.65, 0.71)]


@pytest.mark.parametrize("design,bits,bucket,tile,kind,cap,below,above", LINES, ids=["%s-u%d-b%d-%s" % (c[0], c[1], c[2], c[4]) for c in LINES])
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
