"""Merging tables that never erase: a batch whose hot keys are absent at its start.
Every merge window then finds the same keys missing at the same time; one of them
inserts, the others combine without the lock."""
import numpy as np
import pytest

import oracle
import paper_2509_16407_amd as hw
from paper_2509_16407_amd import workloads as w
from gpu_util import busy_lock_queues, dev, host, per_key_counts, u8

pytestmark = pytest.mark.gpu
FLAGS = hw.F_AGGREGATE | hw.F_NO_ERASE


@pytest.mark.parametrize("design", ["DOUBLE", "DOUBLE_M", "P2", "P2_M", "ICEBERG", "ICEBERG_M", "CHAINING"])
@pytest.mark.parametrize("n,distinct", [(1, 1), (127, 3), (129, 129), (70001, 1), (70001, 40), (300000, 2000)])
def test_hot_keys_absent_at_the_start(design, n, distinct):
    """Windows of one operation, ragged, full; one key, a few, more than a window's
    entries: one DONE per key, every sum exact, in an empty table."""
    t = hw.Table(1 << 14, design, flags=FLAGS)
    om = oracle.OracleMap()
    seed = w.stream_seed(220 + hw.DESIGNS[design], n + distinct)
    pool = w.distinct_keys(seed, distinct)
    k = pool[w.uniform_below(seed + 1, 0, n, distinct)]
    v = w.splitmix64(seed + 2, 0, n)
    st, ost = u8(t.upsert(dev(k), dev(v), combine="sum")), om.upsert(k, v)
    for code in (hw.ST_DONE, hw.ST_EXISTED):
        assert per_key_counts(k, st, code) == per_key_counts(k, ost, code)
    gk, gv = (host(x) for x in t.export())
    o = np.argsort(gk)
    ok, ov = om.dump()
    assert np.array_equal(gk[o], ok) and np.array_equal(gv[o], ov)
    assert busy_lock_queues(t) == 0


@pytest.mark.parametrize("design", ["P2_M", "ICEBERG"])
def test_present_keys_need_no_lock_and_absent_ones_time_out(design):
    """A bucket's lock byte set from the host: its present keys are combined all the
    same, its absent keys report TIMEOUT, all others are written."""
    t = hw.Table(1 << 14, design, flags=FLAGS, lock_timeout_us=1000)
    k = w.distinct_keys(w.stream_seed(230, hw.DESIGNS[design]), 4000)
    v = w.value_of(k)
    assert (u8(t.upsert(dev(k[:2000]), dev(v[:2000]))) == hw.ST_DONE).all()
    home = t.primary_bucket(dev(k)).cpu().numpy()
    b = int(home[3000])
    r = t.raw()
    import torch
    r["locks"].view(torch.uint8)[b * r["lock_stride"]] = 1
    st = u8(t.upsert(dev(k), dev(v)))
    assert (st[:2000] == hw.ST_EXISTED).all()
    late = home[2000:] == b
    assert (st[2000:][late] == hw.ST_TIMEOUT).all() and (st[2000:][~late] == hw.ST_DONE).all()
    f, x = t.query(dev(k[:2000]))
    assert (u8(f) == hw.ST_DONE).all() and np.array_equal(host(x), v[:2000] * np.uint64(2))
