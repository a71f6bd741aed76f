"""Merged mixed calls at the sizes where their windows and the fixed workspace's entry
count change: both entry points against each other, element by element, and
against the oracle's dump."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_16407_amd as hw
from paper_2509_16407_amd import workloads as w
from gpu_util import dev, host, u8

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("distinct", [3, 100000])
@pytest.mark.parametrize("n", [1, 511, 512, 513, 1024, 1025, 4097, 32768, 32769, (1 << 18) - 1, (1 << 18) + 1])
def test_merged_calls_at_window_edges(n, distinct):
    a = hw.Table(1 << 18, "DOUBLE_M", flags=hw.F_MERGE_MIXED)
    b = hw.Table(1 << 18, "DOUBLE_M")
    om = oracle.OracleMap()
    seed = w.stream_seed(280, n + distinct)
    pool = w.distinct_keys(seed, distinct)
    k = pool[w.uniform_below(seed + 1, 0, n, distinct)]
    v = w.splitmix64(seed + 2, 0, n)
    ops = torch.full((n,), hw.OPS["upsert"], dtype=torch.uint8, device="cuda")
    om.upsert(k, v)
    om.upsert(k, v)
    for t, noalloc in ((a, False), (b, n <= 1 << 18)):
        for first in (True, False):
            call = t.mixed_noalloc if noalloc else t.mixed
            st = u8(call(ops, dev(k), dev(v), combine="sum")[0])
            _, lead = np.unique(k, return_index=True)
            if noalloc or t is a:  # the smallest index of a key goes first
                assert (st[lead] == (hw.ST_DONE if first else hw.ST_EXISTED)).all()
            assert (st == hw.ST_DONE).sum() == (len(lead) if first else 0)
            assert (st != hw.ST_DONE).sum() == (st == hw.ST_EXISTED).sum()
        gk, gv = (host(x) for x in t.export())
        o = np.argsort(gk)
        ok, ov = om.dump()
        assert np.array_equal(gk[o], ok) and np.array_equal(gv[o], ov)
