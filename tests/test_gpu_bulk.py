"""Bulk writes grouped by bucket (hw_bulk.hpp) against the CPU oracle: sizes at the
edges of the split (one and two levels, ragged last parts, the smallest grouped
call), every design that has the form, duplicates, reserved keys, skew beyond a
bin's room, tables that have erased, every combine, and a bucket whose lock
another writer holds."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_16407_amd as hw
from paper_2509_16407_amd import workloads as w
from gpu_util import busy_lock_queues, dev, host, image, per_key_counts, u8

pytestmark = pytest.mark.gpu

ODESIGN = {"DOUBLE": oracle.DOUBLE, "DOUBLE_M": oracle.DOUBLE_M, "P2": oracle.P2, "P2_M": oracle.P2_M,
           "ICEBERG": oracle.ICEBERG, "ICEBERG_M": oracle.ICEBERG_M}
CASES = [("DOUBLE", 64, 8, 8), ("DOUBLE_M", 64, 32, 4), ("P2", 64, 32, 8), ("P2_M", 64, 32, 4), ("P2_M", 64, 64, 8),
         ("ICEBERG", 64, 32, 8), ("ICEBERG_M", 64, 32, 4), ("CHAINING", 64, 7, 8), ("DOUBLE", 32, 16, 8),
         ("DOUBLE_M", 32, 32, 4), ("P2", 32, 32, 8), ("P2_M", 32, 32, 8), ("ICEBERG_M", 32, 32, 4)]
IDS = ["%s-u%d-b%d-t%d" % c for c in CASES]


def grouped(t, op, n, combine="sum"):
    return t._scratch(hw.OPS[op], n, hw.COMBINES[combine], None) is not None


def check(t, om):
    k, v = t.export()
    k, v = host(k, t.kv_bits), host(v, t.kv_bits)
    o = np.argsort(k)
    ok, ov = om.dump()
    assert np.array_equal(k[o], ok) and np.array_equal(v[o], ov)
    slots, tags, locks = image(t)
    assert not locks.any() and busy_lock_queues(t) == 0
    if t.design == "CHAINING":
        nv, rep = oracle.chain_check(t.num_buckets, slots.view(np.uint64), locks)
    else:
        nv, rep = oracle.layout_check(ODESIGN[t.design], t.kv_bits, t.num_buckets, t.bucket_slots, slots, tags, locks,
                                      tile_bytes=t.tile * 16)
    assert nv == 0, rep


@pytest.mark.parametrize("design,bits,bucket,tile", CASES, ids=IDS)
@pytest.mark.parametrize("cap", [1 << 12, 1 << 17, 1 << 22])
def test_bulk_ops_against_oracle(design, bits, bucket, tile, cap):
    """Insert to 0.55 and 0.7, insert again (half present), SUM upserts, erase a third
    (with repeats), insert into the erased table, query: 2^12 slots (parts of a few
    buckets), 2^17 (one level) and 2^22 (two levels).  Chaining gets fewer buckets,
    so that chains grow beyond their first node."""
    t = hw.Table(cap if design != "CHAINING" else int(0.7 * cap), design, kv_bits=bits, bucket=bucket, tile=tile)
    om = oracle.OracleMap(key_bits=bits)
    seed = w.stream_seed(170 + hw.DESIGNS[design], bits + bucket)
    n = int(0.7 * cap)
    pool = w.distinct_keys(seed, n + cap // 8, key_bits=bits)
    val = lambda k: w.value_of(k, bits)
    d = lambda a: dev(a, bits)
    cut = int(0.55 * cap) + 5
    assert grouped(t, "insert", cut, "keep") == (not design.startswith("P2")) and grouped(t, "erase", cap // 3 + 4000)
    for k in (pool[:cut], pool[cut:n]):
        assert np.array_equal(u8(t.insert(d(k), d(val(k)))), om.insert(k, val(k)))
    k = np.concatenate([pool[cap // 4: n], pool[n: n + cap // 16 + 3]])
    v = val(k) ^ np.uint64(1)
    assert np.array_equal(u8(t.insert(d(k), d(v))), om.insert(k, v))
    k = np.concatenate([pool[: cap // 3], pool[n + cap // 16 + 3: n + cap // 8]])
    v = (k >> np.uint64(3)) & np.uint64(0xFFFF)
    assert np.array_equal(u8(t.upsert(d(k), d(v), combine="sum")), om.upsert(k, v))
    once = np.concatenate([pool[: cap // 3], w.distinct_keys(seed, 4000, key_bits=bits, skip=len(pool))])
    twice = np.concatenate([once, once[:5000]])
    st, ost = u8(t.erase(d(twice))), om.erase(twice)
    for code in (hw.ST_DONE, hw.ST_MISS):
        assert per_key_counts(twice, st, code) == per_key_counts(twice, ost, code)
    check(t, om)
    k = pool[: cap // 4 + 1]
    assert np.array_equal(u8(t.insert(d(k), d(val(k)))), om.insert(k, val(k)))
    f, x = t.query(d(pool))
    of, ox = om.query(pool)
    assert np.array_equal(u8(f), of) and np.array_equal(host(x, bits), ox)
    check(t, om)


@pytest.mark.parametrize("design,bits,bucket,tile", CASES, ids=IDS)
@pytest.mark.parametrize("combine", ["sum", "min", "max", "keep", "replace"])
def test_bulk_duplicates_reserved_and_skew(design, bits, bucket, tile, combine):
    """As many operations as slots, half of them on one key (more than a bin's room), the
    rest with up to four operations a key, reserved keys in between: statuses per
    key, and the table, equal the oracle's.  Values of one key are equal for REPLACE
    and KEEP, whose result depends on the order."""
    cap = 1 << 16
    t = hw.Table(cap, design, kv_bits=bits, bucket=bucket, tile=tile)
    om = oracle.OracleMap(key_bits=bits)
    seed = w.stream_seed(190 + hw.DESIGNS[design], bits + bucket)
    n = cap
    pool = w.distinct_keys(seed, n // 4, key_bits=bits)
    r = w.uniform_below(seed + 1, 0, n, len(pool))
    k = pool[r]
    k[: n // 2] = pool[7]
    top = (1 << bits) - 1
    k[5::1009] = np.uint64(top)
    k[6::1013] = np.uint64(top - 1)
    k = k[w.permutation(seed + 2, n)]
    v = w.value_of(k, bits) if combine in ("keep", "replace") else w.splitmix64(seed + 3, 0, n) & np.uint64(0xFFFFFFF)
    assert grouped(t, "upsert", n, combine) == (not design.startswith("P2")) and grouped(t, "erase", n)
    code = {"sum": oracle.SUM, "keep": oracle.KEEP, "replace": oracle.REPLACE, "min": oracle.MIN, "max": oracle.MAX}
    st = u8(t.upsert(dev(k, bits), dev(v, bits), combine=combine))
    ost = om.upsert(k, v, combine=code[combine])
    for s in (hw.ST_DONE, hw.ST_EXISTED, hw.ST_INVALID):
        assert per_key_counts(k, st, s) == per_key_counts(k, ost, s)
    check(t, om)
    st, ost = u8(t.erase(dev(k, bits))), om.erase(k)
    for s in (hw.ST_DONE, hw.ST_MISS, hw.ST_INVALID):
        assert per_key_counts(k, st, s) == per_key_counts(k, ost, s)
    check(t, om)


@pytest.mark.parametrize("design", ["DOUBLE_M", "DOUBLE"])
def test_bulk_waits_for_a_held_lock_like_a_plain_call(design):
    """A bucket's lock byte set from the host: the keys of that bucket time out
    without effect, all others are written."""
    cap = 1 << 17
    t = hw.Table(cap, design, lock_timeout_us=1000)
    n = 70001
    k = w.distinct_keys(w.stream_seed(210, hw.DESIGNS[design]), n)
    home = t.primary_bucket(dev(k)).cpu().numpy()
    r = t.raw()
    b = int(home[1000])
    r["locks"].view(torch.uint8)[b * r["lock_stride"]] = 1
    assert grouped(t, "insert", n, "keep")
    st = u8(t.insert(dev(k), dev(w.value_of(k))))
    assert (st[home == b] == hw.ST_TIMEOUT).all() and (st[home != b] == hw.ST_DONE).all()
    f, _ = t.query(dev(k))
    assert np.array_equal(u8(f) == hw.ST_DONE, home != b)


@pytest.mark.parametrize("design,cap", [("ICEBERG_M", 1 << 14), ("DOUBLE", 1 << 13)])
def test_bulk_starts_at_its_smallest_call(design, cap):
    """2048 operations are grouped, 2047 are not, and neither is a call with too few
    operations per slot; the results do not tell."""
    t, om = hw.Table(cap, design), oracle.OracleMap()
    k = w.distinct_keys(w.stream_seed(213, cap), 4095)
    assert hw.BULK_MIN_OPS == 2048
    assert grouped(t, "insert", 2048, "keep") and not grouped(t, "insert", 2047, "keep")
    assert not grouped(hw.Table(1 << 18, design), "insert", 1 << 14, "keep")
    for part in (k[:2048], k[2048:]):
        assert np.array_equal(u8(t.insert(dev(part), dev(w.value_of(part)))),
                              om.insert(part, w.value_of(part)))
    check(t, om)


def test_bulk_status_may_be_left_out_and_scratch_may_be_missing():
    """The C-ABI calls without a status array, and without scratch memory."""
    t = hw.Table(1 << 17, "DOUBLE_M")
    n = 90001
    k = w.distinct_keys(w.stream_seed(211, 1), n)
    dk, dv = dev(k), dev(w.value_of(k))
    sc = t._scratch(hw.OPS["insert"], n, 1, None)
    L, s = hw.lib(), hw._stream(None)
    assert L.hwave_upsert_scratch(t.h, hw._ptr(dk), hw._ptr(dv), n // 2, 1, None, hw._ptr(sc), sc.numel(), s) == 0
    assert L.hwave_upsert_scratch(t.h, hw._ptr(dk), hw._ptr(dv), n, 0, None, None, 0, s) == 0
    f, v = t.query(dk)
    assert bool((f == 1).all())
    twice = np.arange(n) < n // 2
    assert np.array_equal(host(v), np.where(twice, w.value_of(k) * np.uint64(2), w.value_of(k)))
    assert L.hwave_erase_scratch(t.h, hw._ptr(dk), n, None, hw._ptr(sc), sc.numel(), s) == 0
    assert t.size() == 0


@pytest.mark.parametrize("design", ["DOUBLE_M", "DOUBLE", "ICEBERG_M"])
def test_bulk_calls_on_two_streams_at_once(design):
    """Two grouped SUM upserts of the same keys and a grouped insert of others, on
    streams of their own: sums and keys are complete whatever the order."""
    t = hw.Table(1 << 18, design)
    n = 80000
    k = w.distinct_keys(w.stream_seed(212, hw.DESIGNS[design]), 2 * n)
    dk, ones, other = dev(k[:n]), dev(np.ones(n, np.uint64)), dev(k[n:])
    ov = dev(w.value_of(k[n:]))
    torch.cuda.synchronize()
    ss = [torch.cuda.Stream() for _ in range(3)]
    keep = [t.upsert(dk, ones, stream=ss[0]), t.upsert(dk, ones, stream=ss[1]), t.insert(other, ov, stream=ss[2])]
    torch.cuda.synchronize()
    a, b, c = (u8(x) for x in keep)
    assert ((a == 1) ^ (b == 1)).all() and ((a == 2) ^ (b == 2)).all() and (c == 1).all()
    f, v = t.query(dk)
    assert bool((f == 1).all()) and bool((v == 2).all())
    assert t.size() == 2 * n
    check(t, _map(np.concatenate([k[:n], k[n:]]), np.concatenate([np.full(n, 2, np.uint64), w.value_of(k[n:])])))


def test_bulk_call_under_capture_is_the_plain_call():
    """A captured call keeps no scratch memory: replays insert and erase like eager calls."""
    t = hw.Table(1 << 16, "DOUBLE_M")
    n = 30000
    k = w.distinct_keys(w.stream_seed(214, 1), n)
    dk, dv = dev(k), dev(w.value_of(k))
    st, er = torch.empty(n, dtype=torch.uint8, device="cuda"), torch.empty(n, dtype=torch.uint8, device="cuda")
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        assert not grouped(t, "insert", n, "keep")
        t.insert(dk, dv, status=st)
        t.erase(dk, found=er)
    assert grouped(t, "insert", n, "keep")
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
        assert bool((st == hw.ST_DONE).all()) and bool((er == hw.ST_DONE).all()) and t.size() == 0
        assert bool((t.insert(dk, dv) == hw.ST_DONE).all()) and bool((t.erase(dk) == hw.ST_DONE).all())
        st.zero_()
        er.zero_()


def _map(k, v):
    om = oracle.OracleMap()
    om.insert(k, v)
    return om
