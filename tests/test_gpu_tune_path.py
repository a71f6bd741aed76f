"""The tuner times the call that a group's program makes: its rate is that of the same
upserts through Multi.upsert, which are grouped by bucket, not the plain launch's less
than half of it."""
import numpy as np
import pytest
import torch

import paper_2509_16407_amd as hw
from paper_2509_16407_amd import workloads as w
from gpu_util import dev

pytestmark = pytest.mark.gpu


def test_tuned_rate_is_that_of_the_group_call():
    e, load = 14, 0.85
    _, rows = hw.autotune(32, 1 << e, designs=("DOUBLE",), load=load, reps=3)
    row = next(r for r in rows if (r["bucket"], r["tile"]) == (16, 4))
    tables, d = (32 << 20) >> e, int(load * (1 << e))
    k = w.distinct_keys(w.stream_seed(340, 1), d, key_bits=32)
    both = np.empty(2 * d, np.uint64)
    both[0::2], both[1::2] = k, k[w.uniform_below(341, 0, d, d)]
    keys = dev(np.tile(both, tables), 32)
    ts = [hw.Table(1 << e, "DOUBLE", kv_bits=32, bucket=16, tile=4) for _ in range(tables)]
    m = hw.Multi(ts)
    offs = [2 * d * i for i in range(tables + 1)]
    st = torch.empty(keys.numel(), dtype=torch.uint8, device="cuda")
    ms = []
    for _ in range(4):
        m.clear()
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        m.upsert(offs, keys, keys, status=st)
        b.record()
        b.synchronize()
        ms.append(a.elapsed_time(b))
    rate = keys.numel() / min(ms) / 1e6
    print("tuned %.2f, group call %.2f Gops/s" % (row["gops"], rate), flush=True)
    assert 0.6 * rate < row["gops"] < 1.6 * rate
