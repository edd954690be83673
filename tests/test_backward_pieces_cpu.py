"""The piece length that key runs of the backward are cut to: every candidate
tried on the greedy assignment, also those that the planner leaves out because
they cut nothing."""
import heapq

import numpy as np
import pytest

import padoc_synth as syn
import paper_2608_06146_amd as pa


def ceil_div(a, b):
    return -(-a // b)


def piece_blocks(runs, G, Hkv, units):
    """The earliest end over all candidates, the longest pieces on a tie."""
    blocks = [ceil_div(n * G, 32) for n in runs]
    share = ceil_div(sum(blocks) * Hkv, units)
    best = None
    for f in (None, 1.5, 1.2, 0.85, 0.6, 0.42, 0.3, 0.2):
        cap = max(64, max(blocks) if f is None else int(f * share))
        cost, split = [], 0
        for b in blocks:
            pieces = ceil_div(b, cap)
            step = ceil_div(b, pieces)
            split += pieces * Hkv if pieces > 1 else 0
            cost += [ceil_div(min(step, b - x), 2) + 4 for x in range(0, b, step)]
        load = [0] * units
        for c in sorted(cost, reverse=True):
            for _ in range(Hkv):
                heapq.heapreplace(load, load[0] + c)
        end = max(load) + split // 32
        if best is None or end < best[0]:
            best = (end, cap)
    return best[1]


@pytest.mark.parametrize("Hq,Hkv", [(16, 2), (4, 4), (28, 4)])
@pytest.mark.parametrize("tw", [0, 64, 4096])
@pytest.mark.parametrize("shape", ["small pages", "long page", "pages", "one sequence"])
def test_piece_length_is_the_best_candidate(shape, tw, Hq, Hkv):
    rng = np.random.default_rng(len(shape))

    def page(prefix, layout, n, longest):
        f = np.sort(rng.integers(1, layout, n))
        return syn.Page(prefix, prefix, layout, layout, tuple(syn.Branch(int(x), int(y), int(y))
                                                              for x, y in zip(f, rng.integers(1, longest, n))))
    pages = {"small pages": [page(60, 20, 3, 30) for _ in range(40)], "long page": [page(900, 150, 24, 120)],
             "pages": [page(500, 90, 12, 200) for _ in range(4)], "one sequence": [syn.Page(3000, 3000, 10, 10, ())]}[shape]
    segs = pa.segments_from_pages(pages, 0)
    T = syn.count_tokens(pages)
    plan = pa.TreePlan(segs, Hq, Hkv, 64, "bf16", 0, num_kv_rows=T, num_q_rows=int(segs["q_len"].sum()),
                       target_workgroups=tw)
    b = plan.export()["bwd"]
    G = Hq // Hkv
    head0 = b[b["kvh"] == 0]
    runs = {int(r["key_row0"]): int(r["ntok"]) for r in head0}
    cap = piece_blocks(list(runs.values()), G, Hkv, max(1, (tw or 1024) // 4))
    for row0, ntok in runs.items():
        n = ceil_div(ntok * G, 32)
        step = ceil_div(n, ceil_div(n, cap)) * 32
        want = [min(step, ntok * G - c) for c in range(0, ntok * G, step)]
        got = head0[head0["key_row0"] == row0]
        assert sorted(got["ncol"].tolist()) == sorted(want)
