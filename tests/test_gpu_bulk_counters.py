"""Grouped writes as the instrumented library counts them."""
import numpy as np
import pytest

import paper_2509_16407_amd as hw
from paper_2509_16407_amd import workloads as w
from gpu_util import dev, u8

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("design", ["DOUBLE", "DOUBLE_M", "ICEBERG_M", "CHAINING"])
def test_what_is_left_of_a_skewed_call_merges(design):
    """Half of a call on one key, far beyond its bin's room: equal keys of 64 operations
    search under the lock once."""
    t = hw.Table(1 << 15, design, instrumented=True)
    pool = w.distinct_keys(w.stream_seed(290, hw.DESIGNS[design]), 12000)
    n = 24000
    k = pool[np.arange(n) % len(pool)]
    k[::2] = pool[7]
    assert t._scratch(hw.OPS["upsert"], n, 0, None) is not None
    t.insert(dev(pool), dev(np.zeros(len(pool), np.uint64)))
    t.probe_counters(reset=True)
    assert (u8(t.upsert(dev(k), dev(np.ones(n, np.uint64)))) == hw.ST_EXISTED).all()
    assert t.probe_counters()["writes"] <= len(pool) + -(-n // 64)
    f, v = t.query(dev(pool[:12]))
    assert (u8(f) == hw.ST_DONE).all()
    assert v.cpu().tolist() == [int((k == x).sum()) for x in pool[:12]]


@pytest.mark.parametrize("design,load", [("DOUBLE", 0.9), ("DOUBLE_M", 0.95), ("ICEBERG", 0.9), ("ICEBERG_M", 0.9)])
def test_every_distinct_write_is_counted_once(design, load):
    """Grouped inserts, whose claims other parts' keys may take first, and grouped upserts of
    the keys, found in their home bucket or beyond it: one write each, with one
    visit at least."""
    cap = 1 << 18
    t = hw.Table(cap, design, instrumented=True)
    n = int(load * cap)
    k = w.distinct_keys(w.stream_seed(291, hw.DESIGNS[design]), n)
    dk = dev(k)
    assert t._scratch(hw.OPS["insert"], n, 1, None) is not None
    t.probe_counters(reset=True)
    for op, code in (("insert", hw.ST_DONE), ("upsert", hw.ST_EXISTED)):
        assert (u8(getattr(t, op)(dk, dk)) == code).all()
        c = t.probe_counters(reset=True)
        assert c["writes"] == n and c["write_visits"] >= n, (op, c, n)
