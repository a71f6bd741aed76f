"""Grouped iceberg inserts into nearly full tables, and after erases: as few keys end
FULL as in plain calls, a FULL key's buckets are full, and the backyard is filled as
evenly (the standard deviation of its buckets' fills, 12 tables' mean, is that of plain
calls to within five standard errors)."""
import numpy as np
import pytest

import paper_2509_16407_amd as hw
from paper_2509_16407_amd import workloads as w
from gpu_util import dev, full_is_genuine, image, u8

pytestmark = pytest.mark.gpu


def fills(t):
    slots, _, _ = image(t)
    k = slots.view(np.uint64 if t.kv_bits == 64 else np.uint32)[0::2]
    occ = (k < np.uint64((1 << t.kv_bits) - 3)).reshape(t.num_buckets, t.bucket_slots).sum(axis=1)
    return occ[int(0.84 * t.num_buckets):]  # the front yard is the first 83%


@pytest.mark.parametrize("design,bits,bucket,tile", [("ICEBERG", 64, 32, 8), ("ICEBERG_M", 64, 32, 4), ("ICEBERG", 32, 32, 8),
                                                     ("ICEBERG_M", 64, 64, 8)])
@pytest.mark.parametrize("cap,start", [(1 << 15, 0.75), (1 << 18, 0.75), (1 << 18, 0.0), (1 << 20, 0.8), (1 << 20, 0.0)])
@pytest.mark.parametrize("erased", [False, True])
def test_near_full_placement_equals_plain_calls(design, bits, bucket, tile, cap, start, erased, monkeypatch):
    t = hw.Table(cap, design, kv_bits=bits, bucket=bucket, tile=tile)
    grouped = hw.Table._scratch
    n, a, runs = int(0.95 * cap), int(start * cap), 12
    sd, full = {}, {}
    for how in ("plain", "grouped"):
        sd[how], full[how] = [], 0
        for r in range(runs):
            k = w.distinct_keys(w.stream_seed(280 + r, hw.DESIGNS[design]), n + cap // 8, key_bits=bits)
            dk = dev(k, bits)
            monkeypatch.setattr(hw.Table, "_scratch", lambda *x: None)
            t.clear()
            if erased:  # as many keys come and go again
                t.insert(dk[n:].contiguous(), dk[n:].contiguous())
                t.erase(dk[n:].contiguous())
            if a:
                t.insert(dk[:a], dk[:a])
            if how == "grouped":
                monkeypatch.setattr(hw.Table, "_scratch", grouped)
                assert t._scratch(hw.OPS["insert"], n - a, 1, None) is not None
            st = u8(t.insert(dk[a:n], dk[a:n]))
            assert ((st == hw.ST_DONE) | (st == hw.ST_FULL)).all()
            if (st == hw.ST_FULL).any():
                full[how] += int((st == hw.ST_FULL).sum())
                full_is_genuine(t, k[a:n][st == hw.ST_FULL])
            sd[how].append(fills(t).std())
    m = {x: np.mean(v) for x, v in sd.items()}
    se = np.hypot(*[np.std(v, ddof=1) / np.sqrt(runs) for v in sd.values()])
    print("%s u%d b%d 2^%d erased=%d: sd plain %.3f grouped %.3f +- %.3f, FULL %s" % (design, bits, bucket, cap.bit_length() - 1, erased, m["plain"], m["grouped"], se, full), flush=True)
    assert m["grouped"] <= m["plain"] + 5 * se + 0.02
    assert full["grouped"] <= full["plain"] + 5 * np.sqrt(full["plain"] + 1)
