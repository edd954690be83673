"""Private key chunks of a decode plan: 256 keys where chunks of 512 would give
fewer items than target_workgroups, else 512 or more; each key once either way."""
import numpy as np
import pytest

import padoc_synth as syn
import paper_2608_06146_amd as pa


@pytest.mark.parametrize("n_branches,length,target,want", [
    (4, 1000, 0, 256), (4, 200, 0, 256), (255, 1000, 0, 256), (256, 1000, 0, 512), (300, 513, 0, 512),
    (4, 1000, 16, 512), (4, 1000, 17, 256), (1, 1, 0, 256)])
def test_private_chunk_lengths(n_branches, length, target, want):
    br = tuple(syn.Branch(1, length, 1) for _ in range(n_branches))
    segs = pa.segments_from_pages([syn.Page(64, 0, 8, 1, br)], 16)
    nb = int(sum(-(-int(s["len"]) // 16) for s in segs))
    ex = pa.TreePlan(segs, 16, 2, 128, "bf16", 16, num_kv_rows=nb, block_table_len=nb, target_workgroups=target).export()
    priv = ex["work"][ex["n_work_shared"]:]
    n = ex["ranges"]["n_keys"][priv["rng_begin"]]
    assert n.max() == min(length, want)
    # the keys of every branch, once per KV head
    assert n.sum() == 2 * n_branches * length
    r = ex["ranges"][priv["rng_begin"]]
    got = sorted(zip(r["seg"].tolist(), r["key_begin"].tolist(), priv["kvh"].tolist()))
    assert len(got) == len(set(got)) and (np.diff(priv["cost"]) <= 0).all()
