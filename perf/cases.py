"""What a program does with HashWave, as cases whose passes can be timed.

A case is a dict of plain values.  `prepare` makes its state on the GPU from a
seed (keys, values, a resident table, a table group, a server), `run` takes one
pass through the package's public calls, `exact` says what a pass on a fresh
state returns, computed without the package.  The sizes are those of the
benchmark's workloads and of the tests, or generic ones between them.

The kinds of work:

  lookup   read-only queries of a resident table, half of them absent keys
  update   SUM upserts of present keys, then their new values read back
  build    the build and probe sides of a join: clear, insert n distinct keys,
           query all of them and as many absent ones, shuffled
  step     a table's whole life (the load benchmark): clear, inserts in three
           phases, positive and negative queries, SUM upserts, erasing half,
           both query sets again
  churn    one iteration of the aging benchmark: a 1% slice inserted, the oldest
           1% erased, live and absent keys queried, in one mixed launch
  mixed    a skewed batch of queries, SUM upserts and erases in one mixed call
  groupby  many 32-bit tables of uneven capacity, one batched SUM aggregation,
           then every group's sum looked up
  count    a skewed stream counted by key, the counts exported and ordered by key
  serve    requests in pinned host memory served by the continuous batching loop
"""
import math
import random

import torch

import paper_2509_16407_amd as hw

RESERVED = 3  # top key patterns no table accepts


# ------------------------------------------------------------------ inputs

def _mix64(seed, start, count):
    """Elements [start, start + count) of the splitmix64 stream of `seed`, as the
    int64 bit patterns; distinct counters give distinct elements."""
    g = -7046029254386353131  # 0x9E3779B97F4A7C15
    z = torch.arange(start + 1, start + count + 1, dtype=torch.int64, device="cuda")
    z.mul_(g).add_(((int(seed) * 0x5851F42D4C957F2D + 0x14057B7EF767814F) & ((1 << 63) - 1)))
    z = (z ^ ((z >> 30) & ((1 << 34) - 1))).mul_(-4658895280553007687)
    z = (z ^ ((z >> 27) & ((1 << 37) - 1))).mul_(-7723592293110705685)
    return z ^ ((z >> 31) & ((1 << 33) - 1))


def _mix32(seed, start, count):
    """`count` distinct int32 bit patterns: a bijective 32-bit finaliser of a counter."""
    m = 0xFFFFFFFF
    z = torch.arange(start, start + count, dtype=torch.int64, device="cuda")
    z = (z + (int(seed) * 2654435761 + 12345)) & m
    z = (((z ^ (z >> 16)) & m) * 0x7FEB352D) & m
    z = (((z ^ (z >> 15)) & m) * 0x846CA68B) & m
    z = z ^ (z >> 16)
    return torch.where(z >= 1 << 31, z - (1 << 32), z).to(torch.int32)


def _keys(kv, seed, start, count):
    """`count` distinct keys without the reserved top patterns (negative numbers
    close to zero, as signed bit patterns): stream elements from `start` on."""
    z = _mix64(seed, start, count) if kv == 64 else _mix32(seed, start, count)
    bad = (z < 0) & (z >= -RESERVED)
    # a reserved pattern gives way to a stream element past every range in use
    return torch.where(bad, _mix64(seed, 1 << 40, 1) if kv == 64 else _mix32(seed, (1 << 32) - 64, 1), z)


def _value(keys):
    return keys * 3 + 1


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _shuffled(n, seed):
    """A permutation of range(n) as an affine walk (a full sort would cost more than
    the case): tables hash the keys, so only which keys there are matters."""
    a = int(n * 0.6180339887) | 1
    while math.gcd(a, n) != 1:
        a += 2
    return (torch.arange(n, dtype=torch.int64, device="cuda") * a + int(seed) % max(1, n)) % n


class _Zipf:
    """Ranks by the inversion of Gray et al. 1994, theta 0.99."""

    def __init__(self, n, theta=0.99):
        z = sum(float((torch.arange(a, min(n, a + (1 << 24)), dtype=torch.float64, device="cuda") + 1).pow_(-theta).sum())
                for a in range(0, n, 1 << 24))
        self.n, self.theta, self.zeta = n, theta, z
        self.alpha = 1 / (1 - theta)
        self.eta = (1 - (2 / n) ** (1 - theta)) / (1 - (1 + 0.5 ** theta) / z)

    def ranks(self, count, gen):
        u = torch.rand(count, dtype=torch.float64, device="cuda", generator=gen)
        r = (self.n * (self.eta * u - self.eta + 1).pow_(self.alpha)).long().clamp_(max=self.n - 1)
        uz = u * self.zeta
        r = torch.where(uz < 1 + 0.5 ** self.theta, 1, r)
        return torch.where(uz < 1, 0, r)


def _table(case, cap=None, flags=0):
    return hw.Table(cap or case["slots"], case["design"], kv_bits=case["kv"], bucket=case.get("bucket", 0),
                    tile=case.get("tile", 0), flags=flags)


def _elem(case):
    return case["kv"] // 8


# ------------------------------------------------------------------ kinds

class Lookup:
    @staticmethod
    def inputs(case, seed):
        n, total = case["n"], int(case["slots"] * case["load"])
        keys = _keys(case["kv"], seed, 0, total)
        half = n - n // 2
        pos = keys[_shuffled(total, seed)[torch.arange(half, device="cuda") % total]]
        q = torch.cat([pos, _keys(case["kv"], seed, total, n // 2)])
        return keys, q[_shuffled(n, seed + 1)]

    @staticmethod
    def prepare(case, seed):
        keys, q = Lookup.inputs(case, seed)
        t = _table(case)
        t.insert(keys, _value(keys))
        return {"table": t, "q": q}

    @staticmethod
    def run(s):
        found, vals = s["table"].query(s["q"])
        return {"found": found, "values": vals}

    @staticmethod
    def exact(case, seed):
        keys, q = Lookup.inputs(case, seed)
        f = torch.isin(q, keys)
        return {"found": f.to(torch.uint8), "values": torch.where(f, _value(q), 0)}

    @staticmethod
    def work(case):
        return case["n"] * (4 * _elem(case) + 1)


class Update:
    @staticmethod
    def inputs(case, seed):
        total = int(case["slots"] * case["load"])
        keys = _keys(case["kv"], seed, 0, total)
        k = keys[_shuffled(total, seed)[:case["n"]]]
        return keys, k, (_mix64(seed + 1, 0, case["n"]) >> 33).to(k.dtype)

    @staticmethod
    def prepare(case, seed):
        keys, k, v = Update.inputs(case, seed)
        t = _table(case)
        t.insert(keys, _value(keys))
        return {"table": t, "k": k, "v": v}

    @staticmethod
    def run(s):
        status = s["table"].upsert(s["k"], s["v"], combine="sum")
        found, vals = s["table"].query(s["k"])
        return {"status": status, "found": found, "values": vals}

    @staticmethod
    def exact(case, seed):
        _, k, v = Update.inputs(case, seed)
        one = torch.ones_like(k, dtype=torch.uint8)
        return {"status": 2 * one, "found": one, "values": _value(k) + v}

    @staticmethod
    def work(case):
        return case["n"] * (8 * _elem(case) + 2)


class Build:
    @staticmethod
    def inputs(case, seed):
        n = case["n"]
        keys = _keys(case["kv"], seed, 0, n)
        q = torch.cat([keys, _keys(case["kv"], seed, n, n)])[_shuffled(2 * n, seed)]
        return keys, q

    @staticmethod
    def prepare(case, seed):
        keys, q = Build.inputs(case, seed)
        return {"table": _table(case), "keys": keys, "vals": _value(keys), "q": q}

    @staticmethod
    def run(s):
        t = s["table"]
        t.clear()
        status = t.insert(s["keys"], s["vals"])
        found, vals = t.query(s["q"])
        return {"status": status, "found": found, "values": vals}

    @staticmethod
    def exact(case, seed):
        n = case["n"]
        keys, q = Build.inputs(case, seed)
        f = (_shuffled(2 * n, seed) < n)
        return {"status": torch.ones(n, dtype=torch.uint8), "found": f.to(torch.uint8),
                "values": torch.where(f, _value(q), 0)}

    @staticmethod
    def work(case):
        # clear and fill the slots, read the inputs, write the outputs
        e = _elem(case)
        return case["slots"] * 2 * e + case["n"] * (4 * e + 1) + 2 * case["n"] * (4 * e + 1)


class Step:
    FRACTIONS = (0.5 / 0.9, 0.75 / 0.9, 1.0)

    @staticmethod
    def inputs(case, seed):
        n = int(case["slots"] * case["load"])
        q = case["slots"] // 2
        keys = _keys(case["kv"], seed, 0, n)
        walk = _shuffled(n, seed)
        pos = keys[walk[:min(q, n)]]
        neg = _keys(case["kv"], seed, n, min(q, n))
        gone = walk[n - n // 2:]
        return keys, pos, neg, keys[gone], gone

    @staticmethod
    def prepare(case, seed):
        keys, pos, neg, erase, _ = Step.inputs(case, seed)
        ends = [int(f * len(keys)) for f in Step.FRACTIONS]
        vals = _value(keys)
        parts = [(keys[a:b].clone(), vals[a:b].clone()) for a, b in zip([0] + ends[:-1], ends)]
        return {"table": _table(case), "parts": parts, "pos": pos, "neg": neg, "one": torch.ones_like(pos), "erase": erase}

    @staticmethod
    def run(s):
        t = s["table"]
        t.clear()
        out = {"insert": [t.insert(k, v) for k, v in s["parts"]]}
        out["pos"], out["neg"] = t.query(s["pos"]), t.query(s["neg"])
        out["upsert"] = t.upsert(s["pos"], s["one"], combine="sum")
        out["erase"] = t.erase(s["erase"])
        out["pos2"], out["neg2"] = t.query(s["pos"]), t.query(s["neg"])
        return out

    @staticmethod
    def exact(case, seed):
        if case["slots"] > 1 << 24:
            return None
        keys, pos, neg, erase, gone = Step.inputs(case, seed)
        ends = [0] + [int(f * len(keys)) for f in Step.FRACTIONS]
        u8 = lambda n, x: torch.full((n,), x, dtype=torch.uint8)  # noqa: E731
        left = ~torch.isin(pos, erase)
        miss = (u8(len(neg), 0), torch.zeros_like(neg))
        return {"insert": [u8(b - a, 1) for a, b in zip(ends, ends[1:])], "pos": (u8(len(pos), 1), _value(pos)), "neg": miss,
                "upsert": u8(len(pos), 2), "erase": u8(len(erase), 1),
                "pos2": (left.to(torch.uint8), torch.where(left, _value(pos) + 1, 0)), "neg2": miss}

    @staticmethod
    def work(case):
        n, e = int(case["slots"] * case["load"]), _elem(case)
        q = min(case["slots"] // 2, n)
        return case["slots"] * 2 * e + n * (4 * e + 1) + q * (4 * (4 * e + 1) + 5 * e + 1) + n // 2 * (2 * e + 1)


class Churn:
    @staticmethod
    def prepare(case, seed):
        n0 = int(case["slots"] * case["load"])
        s = max(1, n0 // 100)
        n0 = n0 // s * s
        ring = n0 + 12 * s  # keys come back once erased, 11 slices later
        keys = _keys(64, seed, 0, ring)
        absent = _keys(64, seed, ring, s)
        t = _table(case)
        t.insert(keys[:n0], _value(keys[:n0]))
        ops = torch.tensor([1, 3, 0, 0], dtype=torch.uint8, device="cuda").repeat_interleave(s)
        rounds = []
        for i in range(ring // s):
            at = lambda first: keys[(torch.arange(first, first + s, device="cuda")) % ring]  # noqa: E731
            live = i * s + s + (i * 7919 * s) % (n0 - 2 * s)  # a slice that stays through the round
            k = torch.cat([at(n0 + i * s), at(i * s), at(live), absent])
            rounds.append((k, _value(k)))
        return {"table": t, "ops": ops, "rounds": rounds, "i": 0}

    @staticmethod
    def run(s):
        k, v = s["rounds"][s["i"] % len(s["rounds"])]
        s["i"] += 1
        status, vals = s["table"].mixed(s["ops"], k, v)
        return {"status": status, "values": vals}

    @staticmethod
    def exact(case, seed):
        n0 = int(case["slots"] * case["load"])
        s = max(1, n0 // 100)
        n0 = n0 // s * s
        keys = _keys(64, seed, 0, n0 + 12 * s)
        z = torch.zeros(s, dtype=torch.int64, device="cuda")
        st = torch.tensor([1, 1, 1, 0], dtype=torch.uint8).repeat_interleave(s)
        return {"status": st, "values": torch.cat([z, z, _value(keys[s:2 * s]), z])}

    @staticmethod
    def work(case):
        s = max(1, int(case["slots"] * case["load"]) // 100)
        return s * (2 * (4 * 8 + 2) + 2 * (4 * 8 + 2) + 4 * 8)


class Mixed:
    BATCHES = 6

    @staticmethod
    def batches(case, seed):
        """(ops, key ranks, values) per batch: 50% queries, 30% upserts, 20% erases
        over Zipf ranks; a rank has one kind in a batch and is erased at most once,
        so that every query and erase result is the same in any order."""
        n, u = case["n"], case["slots"] // 2
        gen, zipf = _generator(seed), _Zipf(u)
        for b in range(Mixed.BATCHES):
            want = (n - n * 3 // 10 - n // 5, n * 3 // 10, n // 5)
            got = [torch.empty(0, dtype=torch.int64, device="cuda")] * 3
            salt = int(seed) * 64 + b
            while any(len(g) < w for g, w in zip(got, want)):
                r = zipf.ranks(6 * n, gen)
                d = _hash01(r, salt)
                for k, (lo, hi) in enumerate(((0, 0.5), (0.5, 0.8), (0.8, 1.0))):
                    x = torch.cat([got[k], r[(d >= lo) & (d < hi)]])
                    if k == 2:
                        x = torch.unique(x)
                        x = x[_shuffled(len(x), salt)]
                    got[k] = x[:want[k]]
            ranks = torch.cat(got)
            ops = torch.tensor([0, 2, 3], dtype=torch.uint8, device="cuda").repeat_interleave(
                torch.tensor(want, device="cuda"))
            p = torch.randperm(n, device="cuda", generator=gen)
            yield ops[p], ranks[p], _mix64(seed + 17, b * n, n)

    @staticmethod
    def prepare(case, seed):
        u = case["slots"] // 2
        keys = _keys(64, seed, 0, u)
        t = _table(case, flags=0 if case["noalloc"] else hw.F_MERGE_MIXED)
        t.insert(keys, _value(keys))
        return {"table": t, "call": t.mixed_noalloc if case["noalloc"] else t.mixed,
                "batches": [(o, keys[r], v, o != 2) for o, r, v in Mixed.batches(case, seed)], "i": 0}

    @staticmethod
    def run(s):
        ops, k, v, _ = s["batches"][s["i"] % len(s["batches"])]
        s["i"] += 1
        status, vals = s["call"](ops, k, v, combine="sum")
        return {"status": status, "values": vals}

    @staticmethod
    def exact(case, seed):
        keys = _keys(64, seed, 0, case["slots"] // 2)
        ops, r, _ = next(Mixed.batches(case, seed))
        st = torch.where(ops == 2, 2, 1).to(torch.uint8)  # the whole universe is present
        return {"status": st, "values": torch.where(ops == 0, _value(keys[r]), 0)}

    @staticmethod
    def work(case):
        return case["n"] * (1 + 8 + 8 + 9 + 16) + case["n"] * 3 // 10 * 8


def _hash01(r, salt):
    z = (r + salt * 1000003) * -7046029254386353131
    z = (z ^ ((z >> 30) & ((1 << 34) - 1))) * -4658895280553007687
    return ((z >> 33) & ((1 << 30) - 1)).double() / (1 << 30)


class GroupBy:
    @staticmethod
    def inputs(case, seed):
        """Per table D = 0.85 * capacity distinct keys, each once, and as many
        repeats of them, in one shuffled run of 2 D operations."""
        gen, lo, hi = _generator(seed), case["lo"], case["hi"]
        caps = [1 << random.Random(i).randint(lo, hi) for i in range(case["tables"])]  # the case's own, not the seed's
        d = torch.tensor([int(0.85 * c) for c in caps], dtype=torch.int64, device="cuda")
        first = torch.cumsum(d, 0) - d
        total = int(d.sum())
        keys = _keys(32, seed, 0, total)
        mine = torch.repeat_interleave(torch.arange(len(caps), device="cuda"), d, output_size=total)
        repeat = first[mine] + (torch.rand(total, generator=gen, device="cuda", dtype=torch.float64) * d[mine]).long()
        source = torch.stack([torch.arange(total, device="cuda"), repeat], 1).reshape(-1)
        vals = _mix32(seed + 5, 0, 2 * total)
        return caps, [0] + torch.cumsum(d, 0).tolist(), keys, source, vals

    @staticmethod
    def prepare(case, seed):
        caps, ends, keys, source, vals = GroupBy.inputs(case, seed)
        tables = [_table(case, cap=c) for c in caps]
        m = hw.Multi(tables)
        items = [(i, hw.OPS["query"], a, b) for i, (a, b) in enumerate(zip(ends, ends[1:]))]
        return {"multi": m, "offsets": [2 * x for x in ends], "keys": keys[source], "vals": vals, "groups": keys, "items": items}

    @staticmethod
    def run(s):
        m = s["multi"]
        m.clear()
        m.upsert(s["offsets"], s["keys"], s["vals"], combine="sum")
        found, sums = m.run(s["items"], s["groups"])
        return {"found": found, "sums": sums}

    @staticmethod
    def exact(case, seed):
        _, ends, keys, source, vals = GroupBy.inputs(case, seed)
        sums = torch.zeros(len(keys), dtype=torch.int64, device="cuda").index_add_(0, source, vals.long())
        return {"found": torch.ones(len(keys), dtype=torch.uint8), "sums": sums.to(torch.int32)}

    @staticmethod
    def work(case):
        e = case["hi"] - case["lo"] + 1
        slots = case["tables"] * ((1 << case["hi"] + 1) - (1 << case["lo"])) // e
        return slots * 8 + int(0.85 * slots) * (2 * (8 + 1) + 16 + (8 + 9))


class Count:
    @staticmethod
    def inputs(case, seed):
        """Every key of the vocabulary once, the rest of the stream Zipf."""
        u, gen = case["slots"] * 3 // 4, _generator(seed)
        r = torch.cat([torch.arange(u, device="cuda"), _Zipf(u).ranks(case["n"] - u, gen)])
        return _keys(64, seed, 0, u), r[torch.randperm(case["n"], device="cuda", generator=gen)]

    @staticmethod
    def prepare(case, seed):
        keys, r = Count.inputs(case, seed)
        t = _table(case, flags=hw.F_AGGREGATE | hw.F_NO_ERASE)
        return {"table": t, "keys": keys[r], "one": torch.ones_like(r)}

    @staticmethod
    def run(s):
        t = s["table"]
        t.clear()
        t.upsert(s["keys"], s["one"], combine="sum")
        k, c = t.export()
        k, order = torch.sort(k)
        return {"keys": k, "counts": c[order]}

    @staticmethod
    def exact(case, seed):
        keys, r = Count.inputs(case, seed)
        k, c = torch.unique(keys[r], return_counts=True)
        return {"keys": k, "counts": c}

    @staticmethod
    def work(case):
        return case["slots"] * 2 * 16 + case["n"] * (16 + 1) + case["slots"] * 3 // 4 * 16


class Serve:
    @staticmethod
    def requests(case, seed):
        """(table, op, ranks) per request: 50% queries, 30% SUM upserts, 20% inserts.
        Which requests there are is the case's own; their keys come from the seed."""
        u = int(case["slots"] * 0.85)
        zipf, gen = _Zipf(u), _generator(seed)
        own = random.Random(case["requests"])
        for _ in range(case["requests"]):
            a, b, c = own.random(), own.random(), own.random()
            n = int(2 ** (case["lo"] + b * (case["hi"] - case["lo"])))
            op = "query" if c < 0.5 else "upsert" if c < 0.8 else "insert"
            yield int(a * case["tables"]), hw.OPS[op], zipf.ranks(n, gen)

    @staticmethod
    def universe(case, seed, i):
        return _keys(64, seed * 64 + i, 0, int(case["slots"] * 0.85))

    @staticmethod
    def prepare(case, seed):
        tables = []
        for i in range(case["tables"]):
            t = _table(case, flags=hw.F_AGGREGATE | hw.F_NO_ERASE)
            keys = Serve.universe(case, seed, i)
            t.insert(keys, _value(keys))
            tables.append((t, keys))
        torch.cuda.synchronize()
        made = list(Serve.requests(case, seed))
        pad = [(len(r) + 63) // 64 * 64 for _, _, r in made]
        pinned = lambda n, dtype: torch.zeros(n, dtype=dtype, pin_memory=True)  # noqa: E731
        status, out = pinned(sum(pad), torch.uint8), pinned(sum(p for p, m in zip(pad, made) if m[1] == 0), torch.int64)
        requests, at, at_out = [], 0, 0
        for (i, op, r), p in zip(made, pad):
            k = tables[i][1][r]
            q = {"table": i, "op": op, "keys": pinned(len(k), torch.int64).copy_(k), "status": status[at:at + len(k)]}
            if op == hw.OPS["query"]:
                q["out"] = out[at_out:at_out + len(k)]
                at_out += p
            else:
                q["vals"] = pinned(len(k), torch.int64).copy_(_value(k))
            at += p
            requests.append(q)
        return {"server": hw.Server([t for t, _ in tables], slot_ops=1 << 21), "requests": requests, "status": status, "out": out}

    @staticmethod
    def run(s):
        for q in s["requests"]:
            s["server"].submit(**q)
        s["server"].drain()
        return {"status": s["status"], "values": s["out"]}

    @staticmethod
    def exact(case, seed):
        keys = [Serve.universe(case, seed, i) for i in range(case["tables"])]
        held = [_value(k) for k in keys]
        status, out = [], []
        for i, op, r in Serve.requests(case, seed):  # one at a time, in the order of submission
            grow = lambda x: torch.nn.functional.pad(x, (0, -len(x) % 64))  # noqa: E731
            status.append(grow(torch.full((len(r),), 1 if op == hw.OPS["query"] else 2, dtype=torch.uint8)))
            if op == hw.OPS["query"]:
                out.append(grow(held[i][r]))
            elif op == hw.OPS["upsert"]:
                held[i].index_add_(0, r, _value(keys[i][r]))
        return {"status": torch.cat(status), "values": torch.cat(out) if out else torch.zeros(0, dtype=torch.int64)}

    @staticmethod
    def work(case):
        mean = (2 ** case["hi"] - 2 ** case["lo"]) / (math.log(2) * (case["hi"] - case["lo"]))
        return int(case["requests"] * mean * (8 + 16 + 1 + 8))


KINDS = {"lookup": Lookup, "update": Update, "build": Build, "step": Step, "churn": Churn, "mixed": Mixed,
         "groupby": GroupBy, "count": Count, "serve": Serve}


# ------------------------------------------------------------------ cases

def listed():
    return [
        # the smallest request the serving workload draws, looked up in a resident table
        dict(name="lookup_256", kind="lookup", design="P2_M", kv=64, slots=1 << 20, load=0.85, n=256),
        # counters of a few thousand keys raised and read back between other work
        dict(name="update_5000", kind="update", design="DOUBLE_M", kv=64, slots=1 << 20, load=0.8, n=5000),
        # a skewed batch for a caller that cannot allocate
        dict(name="mixed_noalloc_20000", kind="mixed", design="DOUBLE_M", kv=64, slots=1 << 21, n=20000, noalloc=True),
        # the plain double-hashing load test: 943,718 keys into 2^20 slots, then both query sets
        dict(name="build_double_1m", kind="build", design="DOUBLE", kv=64, slots=1 << 20, n=943718),
        # a join on 32-bit keys with an odd number of rows
        dict(name="build_u32_6m", kind="build", design="DOUBLE", kv=32, slots=1 << 23, n=6710887),
        # a table's whole life on the third design family, at the paper's highest load
        dict(name="step_iceberg_2p22", kind="step", design="ICEBERG_M", kv=64, slots=1 << 22, load=0.9),
        # the benchmark's own table, at its full size: the largest case
        dict(name="step_p2m_2p28", kind="step", design="P2_M", kv=64, slots=1 << 28, load=0.85),
        # aging: every kind of operation in one launch on a table at 0.85
        dict(name="churn_p2m_2p24", kind="churn", design="P2_M", kv=64, slots=1 << 24, load=0.85),
        # the benchmark's Zipf batches on its 2^27-slot table
        dict(name="mixed_zipf_1m", kind="mixed", design="DOUBLE_M", kv=64, slots=1 << 27, n=1 << 20, noalloc=False),
        # group-by aggregation over many uneven tables, on the configuration tuning chooses for them
        dict(name="groupby_300_tables", kind="groupby", design="DOUBLE", kv=32, bucket=16, tile=4, tables=300, lo=10, hi=20),
        # counting a skewed stream (words, events) and reading the counts out
        dict(name="count_zipf_4m", kind="count", design="P2_M", kv=64, slots=1 << 21, n=4000000),
        # a burst of requests of uneven sizes over resident tables
        dict(name="serve_burst", kind="serve", design="P2_M", kv=64, slots=1 << 20, tables=16, requests=64, lo=8, hi=17),
    ]


DESIGNS64 = ("DOUBLE", "DOUBLE_M", "P2", "P2_M", "ICEBERG", "ICEBERG_M", "CHAINING", "CUCKOO")
DESIGNS32 = ("DOUBLE", "DOUBLE_M", "P2", "P2_M", "ICEBERG_M")


def _log(rng, lo, hi):
    """A whole number in [lo, hi], spread over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("lookup", "update", "build", "build", "step", "churn", "mixed", "groupby", "count", "serve"))
    kv = rng.choice((64, 64, 32))
    design = rng.choice(DESIGNS64 if kv == 64 else DESIGNS32)
    top = 20 if design == "CUCKOO" else 25
    load = round(rng.uniform(0.4, 0.88), 3)
    if kind in ("lookup", "update"):
        slots = 1 << rng.randint(16, top)
        most = int(slots * load)
        return dict(kind=kind, design=design, kv=kv, slots=slots, load=load, n=_log(rng, 100, min(most, 1 << 23)))
    if kind == "build":
        slots = 1 << rng.randint(12, top)
        return dict(kind=kind, design=design, kv=kv, slots=slots, n=int(slots * load) - rng.randint(0, 9))
    if kind == "step":
        return dict(kind=kind, design=design, kv=kv, slots=1 << rng.randint(14, top), load=load)
    if kind == "churn":
        return dict(kind=kind, design=rng.choice(("P2", "P2_M", "ICEBERG_M", "CHAINING")), kv=64,
                    slots=1 << rng.randint(17, 24), load=min(load, 0.85))
    if kind == "mixed":
        noalloc = rng.random() < 0.5
        n = _log(rng, 1000, 1 << (18 if noalloc else 20))
        lowest = max(16, math.ceil(math.log2(n * 24)))
        return dict(kind=kind, design=rng.choice(("DOUBLE_M", "P2_M", "ICEBERG_M")), kv=64,
                    slots=1 << rng.randint(lowest, max(lowest, 25)), n=n, noalloc=noalloc)
    if kind == "groupby":
        lo = rng.randint(10, 12)
        design, bucket, tile = rng.choice((("DOUBLE", 16, 4), ("DOUBLE", 16, 8), ("DOUBLE_M", 32, 4), ("P2_M", 32, 8)))
        return dict(kind=kind, design=design, kv=32, bucket=bucket, tile=tile, tables=_log(rng, 10, 400), lo=lo,
                    hi=lo + rng.randint(4, 8))
    if kind == "count":
        slots = 1 << rng.randint(14, 22)
        return dict(kind=kind, design=rng.choice(("DOUBLE", "DOUBLE_M", "P2_M", "ICEBERG_M")), kv=64, slots=slots,
                    n=_log(rng, slots, 1 << 23))
    return dict(kind=kind, design=rng.choice(("P2_M", "DOUBLE_M")), kv=64, slots=1 << rng.randint(16, 21),
                tables=rng.randint(2, 24), requests=rng.randint(8, 128), lo=8, hi=rng.randint(12, 18))


# ------------------------------------------------------------------ calls

def prepare(case, seed):
    return dict(KINDS[case["kind"]].prepare(case, seed), kind=case["kind"])


def run(state):
    return KINDS[state["kind"]].run(state)


def exact(case, seed):
    return KINDS[case["kind"]].exact(case, seed)


def work(case):
    return {"bytes": KINDS[case["kind"]].work(case), "flops": 0}
