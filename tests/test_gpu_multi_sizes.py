"""The persistent multi-table launch from one operation to more than the chip's waves
take at once: grids smaller than the chip, chunks of 64 to 256 operations, more
queues than items."""
import numpy as np
import pytest

import paper_2509_16407_amd as hw
from paper_2509_16407_amd import workloads as w
from gpu_util import dev, host, u8

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("designs", [("P2_M",), ("DOUBLE", "P2_M"), ("ICEBERG_M", "DOUBLE_M")], ids="+".join)
@pytest.mark.parametrize("tables,n", [(1, 1), (3, 64), (9, 65), (2, 257), (20, 1000), (7, 30011), (3, 400003)])
def test_every_size_of_launch(designs, tables, n):
    """Insert, query with as many absent keys, erase a third, query: every table of the
    group against the oracle."""
    ts = [hw.Table(max(1 << 12, 2 * n), designs[i % len(designs)]) for i in range(tables)]
    m = hw.Multi(ts)
    pool = w.distinct_keys(w.stream_seed(270, n), 2 * n * tables).reshape(tables, 2 * n)
    run = lambda op, k, v=None: m.run([(i, hw.OPS[op], k.shape[1] * i, k.shape[1] * (i + 1)) for i in range(tables)],
                                      dev(k.reshape(-1)), None if v is None else dev(v.reshape(-1)))
    st, _ = run("insert", pool[:, :n], w.value_of(pool[:, :n].reshape(-1)))
    assert (u8(st) == hw.ST_DONE).all()
    gone = (n + 2) // 3
    for erased in (0, gone):
        if erased:
            st, _ = run("erase", np.ascontiguousarray(pool[:, :erased]))
            assert (u8(st) == hw.ST_DONE).all()
        st, out = run("query", pool)
        there = np.zeros((tables, 2 * n), bool)
        there[:, erased:n] = True
        assert np.array_equal(u8(st).reshape(tables, -1) == hw.ST_DONE, there)
        assert np.array_equal(host(out).reshape(tables, -1)[there], w.value_of(pool[there]))
    assert all(t.size() == n - gone for t in ts)
