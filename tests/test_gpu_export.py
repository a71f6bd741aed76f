"""Export and size over tables whose slot count is below, at and above one block's
share of a pass."""
import numpy as np
import pytest

import paper_2509_16407_amd as hw
from paper_2509_16407_amd import workloads as w
from gpu_util import dev, host, u8

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [64, 32])
@pytest.mark.parametrize("cap,n", [(256, 0), (256, 100), (2048, 1700), (4096, 1), (1 << 16, 40001), (1 << 23, 5000003)])
def test_export_and_size(bits, cap, n):
    t = hw.Table(cap, "DOUBLE", kv_bits=bits)
    k = w.distinct_keys(w.stream_seed(240, cap + bits), n, key_bits=bits)
    v = w.value_of(k, bits)
    if n:
        assert (u8(t.insert(dev(k, bits), dev(v, bits))) == hw.ST_DONE).all()
    assert t.size() == n
    gk, gv = (host(x, bits) for x in t.export())
    o, e = np.argsort(gk), np.argsort(k)
    assert np.array_equal(gk[o], k[e]) and np.array_equal(gv[o], v[e])
