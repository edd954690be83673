"""bf16 tile items whose columns see their first key in a later tile, with
scores far from zero on either side, over row counts that leave a wavefront's
32 result rows full, partly used and unused."""
import math

import numpy as np
import pytest
import torch

import oracle
import padoc_synth as syn
import paper_2608_06146_amd as pa
from _cases import TOL, fill_pool
from oracle import dense as od

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shift", [-300.0, 0.0, 300.0])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads", [(7, 1), (8, 8), (64, 1)])
@pytest.mark.parametrize("q2", [1, 9, 33])
def test_first_key_in_a_later_tile(shift, d, heads, q2):
    """B (fork 0) sees nothing of the root or of A, so its subtree's columns
    have no reference until the item's fifth tile; B's second child sees only 3
    of its keys.  Scores are the drawn ones plus `shift` (log2 units), so
    probabilities relative to 0 would vanish or overflow."""
    Hq, Hkv = heads
    nodes = [(-1, 0, 100, 0), (0, 100, 70, 1), (0, 0, 80, q2), (1, 70, 5, 2), (2, 80, 40, q2), (2, 3, 1, 1)]
    T, nq = sum(n[2] for n in nodes), sum(n[3] for n in nodes)
    scale = 1 / math.sqrt(d)
    q = syn.draw_normal((nq, Hq, d), 5, 1, "bf16", device="cuda")
    k = syn.draw_normal((T, Hkv, d), 5, 2, "bf16", device="cuda")
    v = syn.draw_normal((T, Hkv, d), 5, 3, "bf16", device="cuda")
    q[..., 0] = 16.0
    k[..., 0] = shift / (16.0 * scale * 1.4426950408889634)
    plan = pa.TreePlan(pa.segments_layout(nodes, 0), Hq, Hkv, d, "bf16", 0, num_kv_rows=T, num_q_rows=nq)
    runs = [(pa.tree_attn_fwd(q, k, v, plan), oracle.tree_attention(nodes, q, k, v, scale, Hq, Hkv))]
    n_pool = 60
    kc, vc, ids = fill_pool(nodes, k, v, n_pool, 5)
    O, L = oracle.tree_attention_paged(nodes, q, kc, vc, ids, scale, Hq, Hkv, 16)
    bt = torch.as_tensor(np.asarray(ids), dtype=torch.int32, device="cuda")
    for chunk in (0, 64, 320):
        plan = pa.TreePlan(pa.segments_layout(nodes, 16), Hq, Hkv, d, "bf16", 16, num_kv_rows=n_pool, num_q_rows=nq,
                           block_table_host=np.asarray(ids), max_chunk_keys=chunk)
        runs.append((pa.branch_decode(q, kc, vc, bt, plan), (O, L)))
    torch.cuda.synchronize()
    for (o, lse), (o_ref, l_ref) in runs:
        assert np.abs(o.double().cpu().numpy() - o_ref).max() <= TOL["bf16"][0]
        # scores near 208 (natural units) are summed in fp32: 2^-16 a term, far inside
        assert np.abs(lse.double().cpu().numpy() - l_ref).max() <= TOL["bf16"][0]
