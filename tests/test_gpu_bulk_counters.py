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
