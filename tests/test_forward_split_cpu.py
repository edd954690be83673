"""The packed bf16 schedule with its longest items cut in two, against the one
with every item whole: the same keys for every (token, KV head)."""
import numpy as np
import pytest

import paper_2608_06146_amd as pa

NODES = [(-1, 0, 700, 700), (0, 700, 203, 203), (1, 3, 90, 90), (1, 64, 33, 33), (1, 203, 1, 1), (1, 0, 17, 5),
         (-1, 0, 40, 40), (6, 40, 300, 300)]


def seen(ex, hkv):
    """(token, kvh) -> sorted [(kv_start, keys seen)], and the items' columns."""
    got = {}
    for w in ex["work"]:
        for i in range(w["ntok"]):
            keys = []
            for r in ex["ranges"][w["rng_begin"]:w["rng_begin"] + w["rng_count"]]:
                n = int(r["n_keys"] if r["lim_off"] < 0 else ex["lims"][r["lim_off"] + i])
                assert n <= r["n_keys"] and (r["lim_off"] < 0 or n >= r["min_lim"])
                if n:
                    keys.append((int(r["kv_start"]), n))
            at = (int(ex["toks"][w["tok_begin"] + i]), int(w["kvh"]))
            assert at not in got
            got[at] = sorted(keys)
    return got


@pytest.mark.parametrize("heads", [(16, 2), (28, 4), (1, 1), (64, 1), (8, 8)])
@pytest.mark.parametrize("target", [0, 4, 160, 400, 2048])
def test_cut_items_cover_the_same_keys(heads, target):
    hq, hkv = heads
    segs = pa.segments_layout(NODES, 0)
    T, nq = sum(n[2] for n in NODES), sum(n[3] for n in NODES)

    def plan(t):
        return pa.TreePlan(segs, hq, hkv, 64, "bf16", 0, num_kv_rows=T, num_q_rows=nq, target_workgroups=t).export()

    whole, ex = plan(4), plan(target)  # one compute unit: nothing is cut
    assert seen(ex, hkv) == seen(whole, hkv)
    units, n = (target // 4 or 256), len(whole["work"])
    assert n <= len(ex["work"]) <= max(units, n)
    G = hq // hkv
    wide = {int(k) * G for k in ex["work"]["ntok"]}
    assert max(wide) <= 256
    if n < units and 2 * n <= units:  # room to cut all that are wider than half
        assert max(wide) <= 128 + G
