"""How the bench tells grouped calls from plain ones (CPU only)."""
import bench
import paper_2509_16407_amd as hw


class Table:
    def __init__(self, grouped):
        self.grouped = grouped

    def _scratch(self, op, n, combine, stream):
        return object() if op in self.grouped else None


class Step:
    phase_names = ["insert_0.5", "query_pos", "upsert", "erase", "requery_neg"]
    ops = dict.fromkeys(phase_names, 1 << 20)


def test_phases_name_the_kernels_they_run():
    s = Step()
    s.t = Table({hw.OPS["erase"]})
    k = bench.kernels_of(s)
    assert (k["insert_0.5"], k["query_pos"], k["upsert"], k["erase"]) == ("k_upsert", "k_query", "k_upsert", "grouped_erase")
    ms = {p: [2.0] for p in Step.phase_names}
    ms["erase"] = [9.0]
    assert bench.roofline(ms, s.ops, 1, None, k)["kernel"] == "grouped_erase"


def test_ungrouped_calls_take_no_scratch_memory_and_come_back():
    saved = hw.Table._scratch, hw.Multi._scratch
    with bench.ungrouped():
        assert hw.Table._scratch(None, 0, 1 << 30, 0, None) is None and hw.Multi._scratch(None, [], 1 << 30, 0, None) is None
    assert (hw.Table._scratch, hw.Multi._scratch) == saved
