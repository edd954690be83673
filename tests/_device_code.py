"""The gfx950 code of the built library as instructions, and the wait states
that the hardware asks software for.

The compiler keeps these distances for the instructions it emits.  It does not
look into inline assembly, so they are checked on the disassembly.
"""
import collections
import os
import re
import shutil
import subprocess

import paper_2608_06146_amd as pa

LIB = os.path.join(os.path.dirname(os.path.abspath(pa.__file__)), "libpadoc_attn.so")
OBJDUMP = next((p for p in ("/opt/rocm/llvm/bin/llvm-objdump", shutil.which("llvm-objdump")) if p and os.path.exists(p)), None)

Instr = collections.namedtuple("Instr", "addr op args target")
_LINE = re.compile(r"^\s+([a-z]\w+)\s*(.*?)\s*//\s*([0-9A-Fa-f]+):")
_REG = re.compile(r"\b([sva])(?:(\d+)\b|\[(\d+):(\d+)\])|\b(vcc|m0|exec)\b")
TRANS = ("v_exp_", "v_log_", "v_rcp_", "v_rsq_", "v_sqrt_", "v_sin_", "v_cos_")


def regs(text):
    """Registers an operand names, as (file, index)."""
    out = set()
    for m in _REG.finditer(text):
        if m.group(5):
            out.add((m.group(5), 0))
        elif m.group(2):
            out.add((m.group(1), int(m.group(2))))
        else:
            out.update((m.group(1), i) for i in range(int(m.group(3)), int(m.group(4)) + 1))
    return frozenset(out)


def parse(text):
    """Kernels of a disassembly: name -> list of Instr (`target`: the index a
    branch goes to, or None)."""
    kernels, rows, base = {}, None, 0
    for line in text.splitlines():
        m = re.match(r"^([0-9a-f]+) <(\S+)>:", line)
        if m:
            base = int(m.group(1), 16)
            rows = kernels.setdefault(m.group(2), [])
            continue
        m = _LINE.match(line)
        if m and rows is not None:
            t = re.search(r"<\S+?(?:\+0x([0-9a-f]+))?>\s*$", line)
            to = base + int(t.group(1) or "0", 16) if t and m.group(1).startswith(("s_branch", "s_cbranch")) else None
            rows.append((int(m.group(3), 16), m.group(1), m.group(2), to))
    out = {}
    for name, rs in kernels.items():
        at = {r[0]: i for i, r in enumerate(rs)}
        out[name] = [Instr(a, op, tuple(x.strip() for x in re.split(r",(?![^\[]*\])", args)) if args else (), at.get(to))
                     for a, op, args, to in rs]
    return out


def library_kernels(tmp):
    """Kernels of the built library (its code objects are unbundled into
    directory `tmp`), by mangled name."""
    lib = os.path.join(tmp, "lib.so")
    shutil.copy(LIB, lib)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True, cwd=tmp)
    out = {}
    for f in sorted(os.listdir(tmp)):
        if "gfx950" in f:
            text = subprocess.run([OBJDUMP, "-d", os.path.join(tmp, f)], check=True, capture_output=True, text=True).stdout
            out.update(parse(text))
    return out


def is_valu(op):
    return op.startswith("v_") and not op.startswith(("v_mfma", "v_smfma"))


def is_vmem(op):
    return op.startswith(("global_", "buffer_", "flat_", "scratch_"))


def writes(ins):
    """Registers an ALU instruction writes."""
    if not ins.args:
        return frozenset()
    w = regs(ins.args[0])
    if ins.op.startswith(("v_permlane", "v_swap")) or "_co_" in ins.op:
        w |= regs(ins.args[1])
    if ins.op.startswith("s_cmp") or ins.op.startswith(("s_waitcnt", "s_nop", "s_barrier")):
        return frozenset()
    return w


def reads(ins):
    """Registers an ALU instruction reads."""
    skip = 0 if ins.op.startswith(("v_permlane", "v_swap", "v_fmac", "v_dot2c", "v_mac")) else 1
    return frozenset().union(*[regs(a) for a in ins.args[skip:]]) if ins.args else frozenset()


def wait_states(ins):
    return int(ins.args[0], 0) + 1 if ins.op == "s_nop" else 1


def mfma_states(op):
    """Wait states before a vector instruction may read an MFMA's result
    (32x32x16 and 16x16x32 bf16: 8 and 4 passes; 16x16x4 fp32: 8)."""
    return {"v_mfma_f32_32x32x16_bf16": 12, "v_mfma_f32_16x16x32_bf16": 8, "v_mfma_f32_16x16x4_f32": 10}[op]


def close_pairs(code, reader, writer, need):
    """(writer, reader) instructions closer than need(writer, reader) wait
    states along some path.  reader(ins): the registers that matter or an
    empty set; writer(ins, regs): whether it writes one of them, which ends
    the search on that path."""
    preds = [[] for _ in code]
    for i, ins in enumerate(code):
        if i + 1 < len(code) and ins.op not in ("s_branch", "s_endpgm", "s_setpc_b64"):
            preds[i + 1].append(i)
        if ins.target is not None:
            preds[ins.target].append(i)
    bad = []
    for i, ins in enumerate(code):
        want = reader(ins)
        if not want:
            continue
        todo, seen = [(p, 0) for p in preds[i]], {}
        while todo:
            j, states = todo.pop()
            if states >= 20 or seen.get(j, 99) <= states:
                continue
            seen[j] = states
            w = code[j]
            if writer(w, want):
                if states < need(w, ins):
                    bad.append((w, ins))
                continue
            todo += [(p, states + wait_states(w)) for p in preds[j]]
    return bad


def blocks(code):
    """Basic blocks as (first, last) index pairs with their successors."""
    heads = {0} | {i.target for i in code if i.target is not None}
    heads |= {n + 1 for n, i in enumerate(code) if i.op.startswith(("s_branch", "s_cbranch", "s_endpgm")) and n + 1 < len(code)}
    heads = sorted(heads)
    out = {}
    for a, b in zip(heads, heads[1:] + [len(code)]):
        last = code[b - 1]
        nxt = [] if last.op.startswith(("s_branch", "s_endpgm")) or b == len(code) else [b]
        out[a] = (b, nxt + ([last.target] if last.target is not None else []))
    return out


def loop_blocks(code):
    """Instructions of every block that lies on a cycle."""
    bl = blocks(code)
    reach = {}
    for a in bl:
        seen, todo = set(), list(bl[a][1])
        while todo:
            x = todo.pop()
            if x not in seen:
                seen.add(x)
                todo += bl[x][1]
        reach[a] = seen
    return [code[a:bl[a][0]] for a in bl if a in reach[a]]
