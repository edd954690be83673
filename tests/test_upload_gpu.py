"""Schedules on both sides of the size above which the library's own kernel
copies them (16 KB), and copies read again after the plan was rebuilt in
place: the outputs are those of a resident schedule, bit for bit."""
import numpy as np
import pytest
import torch

import padoc_synth as syn
import paper_2608_06146_amd as pa
from _cases import decode_case, forward_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_branches", [1, 12, 40, 200])
def test_copied_and_resident_schedules_agree(n_branches):
    rng = np.random.default_rng(n_branches)
    br = tuple(syn.Branch(int(f), int(n), 1) for f, n in zip(np.sort(rng.integers(1, 64, n_branches)), rng.integers(1, 90, n_branches)))
    o, lse, plan, (q, kc, vc, bt, ids) = decode_case([syn.Page(130, 0, 64, 1, br)], 16, 2, 128, "bf16", 1, check=False)
    ws = plan.workspace(q.device)
    a, b = torch.empty_like(o), torch.empty_like(lse)
    for _ in range(3):  # the workspace's contents between calls do not matter
        ws.fill_(0x5A)
        pa.branch_decode(q, kc, vc, bt, plan, out=a, lse=b, workspace=ws)
        assert torch.equal(a, o) and torch.equal(b, lse)
    pa.plan_upload(plan, ws)
    pa.branch_decode_resident(q, kc, vc, bt, plan, a, b, ws)
    assert torch.equal(a, o) and torch.equal(b, lse)


def test_forward_with_a_large_schedule():
    """Many short siblings: per-token limits of several hundred KB."""
    rng = np.random.default_rng(2)
    br = tuple(syn.Branch(int(f), 5, 5) for f in np.sort(rng.integers(1, 200, 300)))
    forward_case([syn.Page(64, 64, 200, 200, br)], 28, 4, 64, "bf16", 2, rows=list(range(0, 1764, 97)))
