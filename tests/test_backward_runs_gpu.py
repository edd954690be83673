"""GPU parity of the key-major backward (dK, dV) at the edges of its key
groups (32 keys), runs (128 keys) and column steps (64 columns), of the sums
of split runs, of rows no query sees, and of buffers beyond 4 GB."""
import math

import numpy as np
import pytest
import torch

import padoc_synth as syn
import paper_2608_06146_amd as pa
from _cases import backward_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 31, 32, 33, 64, 65, 127, 128, 129, 257])
@pytest.mark.parametrize("heads,d", [((1, 1), 128), ((7, 1), 64), ((16, 2), 128), ((64, 1), 64)])
def test_run_and_step_edges(n, heads, d):
    """A root of n keys; below it 1, 3 and 9 query tokens that see all, some
    and one of them (1 to 13 * G columns)."""
    nodes = [(-1, 0, n, min(n, 2)), (0, n, 1, 1), (0, (n + 1) // 2, 3, 3), (0, 1, 9, 9)]
    backward_case(nodes, heads[0], heads[1], d, n)


@pytest.mark.parametrize("d", [64, 128])
def test_split_runs_are_summed_in_order(d):
    """Runs cut into several pieces: parity, and the same bits twice."""
    rng = np.random.default_rng(d)
    br = tuple(syn.Branch(int(f), int(n), int(n)) for f, n in zip(np.sort(rng.integers(1, 97, 40)), rng.integers(20, 90, 40)))
    pages = [syn.Page(300, 300, 96, 96, br)]
    errs, plan = backward_case(pages, 16, 2, d, 5)
    b = plan.export()["bwd"]
    assert (b["ncol"] < b["ntok"] * 8).any(), "expected split key runs"
    first, _ = backward_case(pages, 16, 2, d, 5, check=False)
    again, _ = backward_case(pages, 16, 2, d, 5, check=False)
    assert all(torch.equal(x, y) for x, y in zip(first, again))


@pytest.mark.parametrize("scale", [1e-35, 1e-37, 2e-38, 1.2e-38])
def test_scales_at_which_lse_over_scale_leaves_fp32(scale):
    """LSE / scale, from which dK/dV's scores start, passes 3.4e38 at the
    smallest scales a plan takes; the probabilities are those of a plain mean.
    Tolerance: P and the result are bf16 (2^-9 each, relative) on sums of n
    terms of rms 1/i."""
    n, d = 150, 128
    q, k, v, do = (syn.draw_normal((n, 2, d), 11, i, "bf16", device="cuda") for i in range(4))
    segs = pa.segments_layout([(-1, 0, n, n)], 0)
    plan = pa.TreePlan(segs, 2, 2, d, "bf16", 0, softmax_scale=scale, num_kv_rows=n, num_q_rows=n)
    o, lse = pa.tree_attn_fwd(q, k, v, plan)
    assert torch.allclose(lse.double().cpu(), torch.arange(1, n + 1).double().log()[:, None].expand(n, 2), atol=1e-5)
    dq, dk, dv = pa.tree_attn_bwd(q, k, v, o, lse, do, plan)
    torch.cuda.synchronize()
    P = torch.ones(n, n, dtype=torch.float64).tril() / torch.arange(1, n + 1)[:, None]
    want = torch.einsum("ij,ihd->jhd", P, do.double().cpu())
    err = (dv.double().cpu() - want).norm() / want.norm()
    assert err < 2 ** -8, float(err)
    assert all(bool(torch.isfinite(g).all()) for g in (dq, dk))


def test_rows_without_queries_are_zero():
    """Gaps between segments, and keys that no query sees, get zero gradients
    whatever the buffers held."""
    Hq, Hkv, d = 8, 2, 128
    nodes = [(-1, 0, 150, 20), (0, 0, 40, 40), (0, 100, 30, 0)]  # rows 0..129 are seen by the last 20 tokens only
    segs = pa.segments_layout(nodes, 0)
    off, at = [], 3
    for n in nodes:
        off.append(at)
        at += n[2] + 5
    segs["kv_off"] = off
    T, nq = at, 60
    q, k, v, do = (syn.draw_normal(s, 7, i, "bf16", device="cuda")
                   for i, s in enumerate([(nq, Hq, d), (T, Hkv, d), (T, Hkv, d), (nq, Hq, d)]))
    plan = pa.TreePlan(segs, Hq, Hkv, d, "bf16", 0, num_kv_rows=T, num_q_rows=nq)
    o, lse = pa.tree_attn_fwd(q, k, v, plan)
    dk, dv = torch.full_like(k, 9.0), torch.full_like(v, 9.0)
    print("[case] backward rows without queries", flush=True)
    pa.tree_attn_bwd(q, k, v, o, lse, do, plan, dk=dk, dv=dv)
    torch.cuda.synchronize()
    seen = torch.zeros(T, dtype=torch.bool)
    seen[off[0]:off[0] + 150] = True
    seen[off[1]:off[1] + 40] = True
    for g in (dk, dv):
        assert bool((g[~seen.cuda()] == 0).all())
        assert bool((g[seen.cuda()].float().abs().amax(dim=(1, 2)) > 0).all())


def test_rows_beyond_four_gigabytes():
    """Queries past the first 4 GB of Q: the last pages' gradients equal those
    of the pages on their own."""
    Hq, Hkv, d, n = 64, 1, 128, 30  # 1,920 columns: never split, so bit for bit the same
    pages = 4 * (1 << 30) // (n * Hq * d * 2) + 40
    nodes = [(-1, 0, n, n)] * pages
    T = n * pages
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    q, do = (torch.randn((T, Hq, d), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    k, v = (torch.randn((T, Hkv, d), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    print(f"[case] backward beyond 4 GB: {pages} pages of {n} tokens, Hq={Hq}", flush=True)

    def run(pages, q, k, v, do):
        plan = pa.TreePlan(pa.segments_layout([(-1, 0, n, n)] * pages, 0), Hq, Hkv, d, "bf16", 0, num_kv_rows=k.shape[0],
                           num_q_rows=q.shape[0])
        o, lse = pa.tree_attn_fwd(q, k, v, plan)
        return pa.tree_attn_bwd(q, k, v, o, lse, do, plan)

    whole = run(pages, q, k, v, do)
    for part in (slice(0, 20 * n), slice(T - 20 * n, T)):
        alone = run(20, q[part].contiguous(), k[part].contiguous(), v[part].contiguous(), do[part].contiguous())
        for a, b in zip(whole, alone):
            assert torch.equal(a[part], b)
