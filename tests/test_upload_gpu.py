"""Schedules on both sides of the size above which the library's own kernel
copies them (16 KB): the outputs are those of a resident schedule, bit for
bit; and host copies that are written again for the next step while the GPU is
behind (a plan rebuilt in place, a session's staging buffers): the outputs are
those of steps that wait for one another."""
import ctypes as C

import numpy as np
import pytest
import torch

import padoc_synth as syn
import paper_2608_06146_amd as pa
from paper_2608_06146_amd import _lib
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


HQ, HKV, D, ROOTS, STREAMS = 16, 4, 128, 4, 400


def _forked_session(seed):
    """Four prefixes of 200 tokens and 100 streams off each, 3 to 10 tokens
    long, over a pool whose every slot holds a value (so that later tokens need
    no rows written: a step's K/V are the pool's)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    n = 800
    kc = torch.randn(n, HKV, D // 8, 16, 8, device="cuda", generator=g).bfloat16()
    vc = torch.randn(n, HKV, D, 16, device="cuda", generator=g).bfloat16()
    bt = torch.zeros(8192, dtype=torch.int32, device="cuda")
    s = pa.DecodeSession(HQ, HKV, D, n, "bf16", k_cache=kc, v_cache=vc, block_table=bt)
    rows = [torch.randn(10 * STREAMS, HKV, D, device="cuda", generator=g).bfloat16() for _ in "kv"]

    def prefill(n_new):
        n_new = np.asarray(n_new)
        s.step(None, rows[0][:n_new.sum()], rows[1][:n_new.sum()], n_new, 0 * n_new)

    roots = [s.open() for _ in range(ROOTS)]
    prefill([200] * ROOTS)
    for i in range(STREAMS):
        s.open(roots[i % ROOTS], 200 - i // ROOTS)
    for r in roots:
        s.close(r)
    prefill(3 + np.arange(STREAMS) % 8)
    return s


def _steps():
    """Query rows of each step: from few streams to all (the schedules, and the
    buffers that hold them, grow), and fewer again."""
    rng = np.random.default_rng(5)
    for count in (200, 250, 400, 300, 400, 220):
        n = np.zeros(STREAMS, np.int32)
        n[rng.permutation(STREAMS)[:count]] = 1
        yield n


def _run(mode, wait):
    s = _forked_session(3)
    g = torch.Generator(device="cuda").manual_seed(9)
    q = torch.randn(STREAMS, HQ, D, device="cuda", generator=g).bfloat16()
    kv = torch.randn(2, STREAMS, HKV, D, device="cuda", generator=g).bfloat16()
    busy = torch.ones(8192, 8192, dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    outs = []
    torch.cuda.synchronize()
    if not wait:  # about 10 ms ahead of the first step
        for _ in range(12):
            busy @ busy
    for n in _steps():
        nk, nq, need = s.prepare(n, n)
        v = s.view(schedule=True, block_table=False)
        assert need <= ws.numel() and sum(v["schedule"][k].nbytes for k in ("work", "ranges", "lims", "toks")) > 16384
        o, lse = torch.empty_like(q[:nq]), torch.empty(nq, HQ, device="cuda")
        if mode == "session":
            s.launch(q[:nq], kv[0, :nk], kv[1, :nk], out=o, lse=lse, workspace=ws)
        else:  # the step's plan, as a caller that appends its own rows runs it
            assert len(v["patch"]) == 0
            _lib.check(_lib.lib().padoc_branch_decode(
                C.c_void_p(v["plan"]), *[C.c_void_p(t.data_ptr()) for t in (q, s.k_cache, s.v_cache, s.block_table, o, lse, ws)],
                ws.numel(), C.c_void_p(torch.cuda.current_stream().cuda_stream)))
            s.commit()
        if wait:
            torch.cuda.synchronize()
        outs += [o, lse]
    torch.cuda.synchronize()
    assert all(bool(torch.isfinite(t).all()) for t in outs)
    return outs


@pytest.mark.parametrize("mode", ["session", "plan"])
def test_host_copies_written_again_while_the_gpu_is_behind(mode):
    print(f"[case] steps back to back, {mode}", flush=True)
    want = _run(mode, wait=True)
    assert all(torch.equal(a, b) for a, b in zip(_run(mode, wait=False), want))
