"""Wait states between the instructions of the kernels that are partly written in assembly: the compiler keeps them between
its own instructions, but does not look inside an assembly statement.  The kernels are compiled to assembly with the
build's flags and every path through them is followed, with the rules of the gfx940 family that such code can break."""
import os
import re
import subprocess

import pytest

from paper_2401_09149_amd import build

TRANS = ("v_exp", "v_log", "v_rcp", "v_rsq", "v_sqrt")
# What an instruction leaves behind -> wait states until a register may be used.  VCC and scalar registers written by a
# VALU instruction are read by VALU instructions 2 later, transcendental results by other VALU instructions 1 later.
# MFMAs and half-wave swaps read what other VALU instructions wrote 2 later.  A register that an MFMA of four or eight passes takes as its C operand may be written by VALU 3 or 7 later, its result
# be used (by other than the next MFMA of its chain) 8 or 12 later.  An MFMA is held back until the one in front of it has
# gone through its passes.
READ_BY_VALU = {"scalar": 2, "trans": 1}
READ_BY_MFMA = 2
C_OPERAND = {4: 3, 8: 7}
RESULT = {4: 8, 8: 12}
KEEP = 24   # longer than any rule


def regs(op):
    op = op.strip().lstrip("-|")
    m = re.match(r"([vas])\[(\d+):(\d+)\]", op)
    if m:
        return {(m[1], i) for i in range(int(m[2]), int(m[3]) + 1)}
    m = re.match(r"([vas])(\d+)\b", op)
    return {(m[1], int(m[2]))} if m else {("vcc", 0)} if op.startswith("vcc") else set()


class Instruction:
    def __init__(self, line):
        self.text = line
        self.op, _, rest = line.partition(" ")
        ops = [o.strip() for o in rest.split(",")] if rest else []
        self.states = int(ops[0], 0) + 1 if self.op == "s_nop" else 1
        self.valu = self.op.startswith("v_")
        self.mfma = self.op.startswith("v_mfma")
        self.passes = 4 if "16x16x32" in self.op else 8
        self.memory = self.op.startswith(("ds_", "global_", "flat_", "buffer_"))
        self.trans = self.op.startswith(TRANS)
        self.target = ops[0] if self.op.startswith(("s_branch", "s_cbranch")) else None
        self.ends = self.op in ("s_branch", "s_endpgm", "s_setpc_b64")
        self.reads, self.writes, self.c = set(), set(), set()
        if self.memory:
            self.reads = set().union(*map(regs, ops))
        if self.valu:
            two = self.op.startswith(("v_permlane16_swap", "v_permlane32_swap", "v_swap")) or re.match(
                r"v_(add|sub|subrev|addc|subb)_co|v_mad_[ui]64|v_div_scale", self.op)
            n = 2 if two else 1
            self.writes = set().union(*map(regs, ops[:n]))
            self.c = regs(ops[3]) if self.mfma else set()
            self.reads = set().union(*map(regs, ops[n:])) - self.c
            if self.op.startswith(("v_permlane", "v_swap", "v_fmac", "v_dot2c")):
                self.reads |= self.writes
            if self.op.startswith(("v_cndmask_b32_e32", "v_div_fmas")):
                self.reads.add(("vcc", 0))


def parse(path):
    """name -> (instructions, label -> index) of every kernel in an assembly listing."""
    kernels, code = {}, None
    for raw in open(path):
        line = " ".join(raw.split(";")[0].split())
        m = re.match(r"(_Z\w+):", line)
        if m:
            code, labels = [], {}
            kernels[m[1]] = (code, labels)
        elif line.startswith(".Lfunc_end"):
            code = None
        elif code is not None and line.endswith(":"):
            labels[line[:-1]] = len(code)
        elif code is not None and line and not line.startswith("."):
            code.append(Instruction(line))
    return kernels


def step(i, state, faults):
    """What is pending behind instruction `i`; state: (kind, register) -> wait states since it was written."""
    if i.mfma:
        held = max([passes - state.get(("matrix core", passes), KEEP) for passes in (4, 8)] + [0])
        state = {k: age + held for k, age in state.items()}
    def need(kind, registers, states):
        for r in registers:
            if state.get((kind, r), KEEP) < states:
                faults.add((str(kind), i.text, state[kind, r]))
    for passes in (4, 8):
        if i.valu or i.memory:
            need(("result", passes), i.reads, RESULT[passes])
        if i.valu and not i.mfma:
            need(("result", passes), i.writes, RESULT[passes])
            need(("c operand", passes), i.writes, C_OPERAND[passes])
    if i.mfma or i.op.startswith("v_permlane"):
        need("vector", i.reads | i.c, READ_BY_MFMA)
    if i.valu:
        need("scalar", i.reads, READ_BY_VALU["scalar"])
        if not i.trans and not i.mfma:
            need("trans", i.reads, READ_BY_VALU["trans"])
    state = {k: age + i.states for k, age in state.items() if age + i.states < KEEP and (k[1] not in i.writes or k[0][0] == "c operand")}
    if i.mfma:
        state["matrix core", i.passes] = 0
    for r in i.c:
        state[("c operand", i.passes), r] = 0
    for r in i.writes if i.valu else ():
        if r[0] in ("s", "vcc"):
            state["scalar", r] = 0
        elif i.mfma:
            state[("result", i.passes), r] = 0
        else:
            state["vector", r] = 0
            if i.trans:
                state["trans", r] = 0
    return state


def check(code, labels):
    starts = sorted({0, *labels.values()} | {n + 1 for n, i in enumerate(code) if i.target or i.ends})
    ends = dict(zip(starts, starts[1:] + [len(code)]))
    faults, entry, todo = set(), {0: {}}, [0]
    while todo:
        n = todo.pop()
        state, follow = dict(entry[n]), []
        for i in code[n:ends[n]]:
            state = step(i, state, faults)
            if i.target:
                follow.append(labels[i.target])
        if ends[n] < len(code) and not (ends[n] > n and code[ends[n] - 1].ends):
            follow.append(ends[n])
        for f in follow:   # the shortest distance over all ways in (and the matrix core idle for longest)
            old = entry.get(f)
            new = {k: age for k, age in (state if old is None else old).items() if k[0] != "matrix core" or k in state}
            for k, age in state.items():
                if k[0] == "matrix core":
                    if k in new:
                        new[k] = max(age, new[k])
                else:
                    new[k] = min(age, new.get(k, KEEP))
            if new != old:
                entry[f] = new
                todo.append(f)
    return faults


@pytest.mark.parametrize("src", ["attn_fwd.hip", "attn_fwd_wide.hip", "attn_bwd.hip", "linear_gemm.hip"])
def test_no_instruction_reads_a_register_too_early(src, tmp_path):
    out = str(tmp_path / "kernels.s")
    flags = [f for f in build.FLAGS if not f.startswith("-Rpass")] + build.SOURCE_FLAGS.get(src, [])
    subprocess.run(["hipcc", *flags, "--cuda-device-only", "-S", os.path.join(build.CSRC, src), "-o", out], check=True,
                   capture_output=True)
    kernels = parse(out)
    assert any(i.mfma for code, _ in kernels.values() for i in code)
    for name, (code, labels) in kernels.items():
        faults = check(code, labels)
        assert not faults, (name, len(faults), sorted(faults)[:4])
