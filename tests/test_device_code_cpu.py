"""Wait states of the built kernels, on their disassembly.

Inline assembly (the direct global -> LDS loads, v_max3_f32) is opaque to the
compiler, which otherwise keeps these distances: no pair of instructions may
be closer than the hardware asks for, along any path.
"""
import pytest

import _device_code as dc

NONE = frozenset()


def _valu_writer(w, r):
    return w.op.startswith("v_") and bool(dc.writes(w) & r)


# hazard: (reader's registers, writes one of them, wait states needed)
HAZARDS = {
    "M0 written by the scalar unit, then a load to LDS": (
        lambda i: frozenset([("m0", 0)]) if "_lds_" in i.op else NONE,
        lambda w, r: bool(dc.writes(w) & r), lambda w, r: 1),
    "SGPR written by a vector instruction, then read by a memory instruction": (
        lambda i: frozenset(x for a in i.args for x in dc.regs(a) if x[0] in ("s", "vcc")) if dc.is_vmem(i.op) else NONE,
        lambda w, r: bool(dc.writes(w) & r), lambda w, r: 5 if dc.is_valu(w.op) else 0),
    "VGPR written by a vector instruction, then read by a lane swap": (
        lambda i: dc.reads(i) if i.op.startswith("v_permlane") else NONE, _valu_writer, lambda w, r: 2),
    "transcendental result, then read by another vector instruction": (
        lambda i: dc.reads(i) if dc.is_valu(i.op) and not i.op.startswith(dc.TRANS) else NONE, _valu_writer,
        lambda w, r: 1 if w.op.startswith(dc.TRANS) else 0),
    "matrix product, then read by a vector instruction": (
        lambda i: dc.reads(i) if dc.is_valu(i.op) else NONE, _valu_writer,
        lambda w, r: dc.mfma_states(w.op) if w.op.startswith("v_mfma") else 0),
}


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if dc.OBJDUMP is None:
        pytest.skip("llvm-objdump not found")
    k = dc.library_kernels(str(tmp_path_factory.mktemp("code")))
    assert sum("bwd_dkdv" in n for n in k) == 4 and sum("tile_mfma_bf16" in n for n in k) == 2
    return k


@pytest.mark.parametrize("hazard", HAZARDS)
def test_wait_states(kernels, hazard):
    bad = {n: p[0] for n, c in kernels.items() if (p := dc.close_pairs(c, *HAZARDS[hazard]))}
    assert not bad, bad


def test_no_packed_fp32(kernels):
    assert not [(n, i) for n, c in kernels.items() for i in c if i.op in ("v_pk_add_f32", "v_pk_mul_f32", "v_pk_fma_f32")]


# Each hazard, one wait state short and just far enough; the branch makes the
# short distance one around a loop.
SHORT = {
    "M0 written by the scalar unit, then a load to LDS": (
        "s_mov_b32 m0, s4", "global_load_lds_dwordx4 v1, s[2:3]", 1),
    "SGPR written by a vector instruction, then read by a memory instruction": (
        "v_readfirstlane_b32 s3, v7", "global_load_dword v1, v0, s[2:3]", 5),
    "VGPR written by a vector instruction, then read by a lane swap": (
        "v_max3_f32 v3, v4, v5, v6", "v_permlane32_swap_b32_e32 v2, v3", 2),
    "transcendental result, then read by another vector instruction": (
        "v_exp_f32_e32 v3, v4", "v_add_f32_e32 v1, v2, v3", 1),
    "matrix product, then read by a vector instruction": (
        "v_mfma_f32_32x32x16_bf16 v[16:31], v[0:3], v[4:7], v[16:31]", "v_max3_f32 v1, v2, v30, v31", 12),
}


@pytest.mark.parametrize("loop", [False, True])
@pytest.mark.parametrize("hazard", HAZARDS)
def test_the_check_sees_a_missing_state(hazard, loop):
    first, second, need = SHORT[hazard]
    for states in (need - 1, need):
        nops = ["s_nop 0"] * states
        if loop and not states:
            continue
        if loop:  # the reader stands before the writer; the branch is one of the states
            lines = [second, first] + nops[1:] + ["s_cbranch_scc0 65530 <k>"]
        else:
            lines = [first] + nops + [second]
        text = "0000000000000100 <k>:\n" + "".join(
            f"\t{x.split(' <')[0]}    // {0x100 + 8 * i:012X}: 00000000{' <k>' if '<k>' in x else ''}\n"
            for i, x in enumerate(lines + ["s_endpgm"]))
        pairs = dc.close_pairs(dc.parse(text)["k"], *HAZARDS[hazard])
        assert bool(pairs) == (states < need), (text, pairs)


# Kernels whose loops keep loads to LDS in flight across steps, at counts they
# wait for themselves: the wait at each such loop's barrier is the only one.
@pytest.mark.parametrize("kernel", ["tile_mfma_bf16", "bwd_dq", "bwd_dkdv"])
def test_steps_do_not_drain_the_loads_in_flight(kernels, kernel):
    """In a loop with loads to LDS, a block waits for vector memory only right
    before a barrier, or behind a load of its own into registers (the limits of
    the next key range)."""
    found = 0
    for name, code in kernels.items():
        if kernel not in name:
            continue
        for block in dc.loop_blocks(code):
            found += any("_lds_" in i.op for i in block)
            for n, i in enumerate(block):
                if i.op != "s_waitcnt" or "vmcnt" not in " ".join(i.args):
                    continue
                at = code.index(i)
                # (a branch around a wavefront's wait for its own LDS stores may stand between)
                own = any(x.op.startswith("global_load") and "_lds_" not in x.op for x in code[at - 8:at])
                assert own or any(x.op == "s_barrier" for x in code[at:at + 5]), (name, i)
    assert found >= 2
