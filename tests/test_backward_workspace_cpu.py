"""The backward workspace: room for what the kernels keep there, and no more."""
import pytest

import paper_2608_06146_amd as pa


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("nodes", [
    [(-1, 0, 100, 100)] * 300,  # pages of their own: no run is split
    [(-1, 0, 1500, 0), (0, 1500, 2000, 2000)],  # a prefix that 2,000 tokens see: split runs
])
def test_holds_the_slots_and_the_lists(nodes, d):
    Hq, Hkv = 32, 4
    T, nq = sum(n[2] for n in nodes), sum(n[3] for n in nodes)
    plan = pa.TreePlan(pa.segments_layout(nodes, 0), Hq, Hkv, d, "bf16", 0, num_kv_rows=T, num_q_rows=nq)
    ex = plan.export()
    b = ex["bwd"]
    slots = int((b["ncol"] < b["ntok"] * (Hq // Hkv)).sum())
    assert (slots > 0) == (len(nodes) == 2)
    part = max(1, slots) * 2 * 128 * d * 4
    # two values per query row and head; query row and limit per listed token
    lists = 2 * nq * Hq * 4 + 2 * len(ex["btoks"]) * 4
    # the schedules' records as exported, each section and record at most
    # doubled by padding and the compact lists
    records = sum(ex[k].nbytes for k in ("work", "ranges", "lims", "toks", "bwd"))
    nb = plan.backward_workspace_bytes()
    assert part + lists <= nb <= part + lists + 2 * records + (1 << 16), (nb, part, lists, records)
