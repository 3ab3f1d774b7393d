"""The pipelined attention kernels write their MFMAs as inline assembly and keep every value in a register of its own.  The
compiler knows nothing of the wait states between such an MFMA and the vector instructions around it: with a spilled or
moved operand, or a vector instruction placed too close, they are gone.  Compiles the kernels (no GPU needed)."""
import os
import re
import subprocess

import pytest

from paper_2603_21257_amd import build as b

# Wait states (instructions, s_nop n as n + 1): a vector instruction's result before an MFMA reads it; a 16x16x32 bf16 MFMA's
# result before anything but the accumulation into it reads or writes it.
BEFORE, AFTER = 2, 11


def regs(text):
    out = set()
    for k, lo, hi, n in re.findall(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        out |= {k + str(i) for i in (range(int(lo), int(hi) + 1) if lo else [int(n)])}
    return out


class Ins:
    """One instruction: vector registers read and written, wait states that it takes."""

    def __init__(self, line):
        self.line = line
        self.op, _, rest = line.partition(" ")
        ops = re.split(r",\s*(?![^\[]*\])", rest.strip()) if rest.strip() else []
        self.mfma = self.op.startswith("v_mfma")
        self.vector = self.op.startswith("v_")
        memory_load = re.match(r"(ds_read|ds_bpermute|ds_permute|ds_swizzle|global_load|flat_load|buffer_load|scratch_load)", self.op)
        if re.match(r"v_(cmp|readlane|readfirstlane)", self.op) or "load_lds" in self.op:
            dst = []
        elif re.match(r"v_(permlane\d+_swap|swap)", self.op):
            dst = ops[:2]
        else:
            dst = ops[:1] if self.vector or memory_load else []
        self.writes = set().union(*map(regs, dst))
        reads = ops if len(dst) == 2 or not dst else ops[1:]
        self.reads = set().union(*map(regs, reads))
        self.states = int(ops[0], 0) + 1 if self.op == "s_nop" else 1


class Code:
    """Instructions of one kernel with the edges between them."""

    def __init__(self, asm, kernel):
        body = re.search(r"^(\w*%s\w*):[^\n]*\n(.*?)^\.Lfunc_end" % kernel, asm, re.M | re.S).group(2)
        self.ins, at, jumps = [], {}, []
        for line in body.splitlines():
            line = re.sub(r"\s+", " ", line.split(";")[0].split("//")[0]).strip()
            if line.endswith(":"):
                at[line[:-1]] = len(self.ins)
            elif line and not line.startswith("."):
                self.ins.append(Ins(line))
        self.succ = []
        for i, x in enumerate(self.ins):
            go = [] if x.op in ("s_endpgm", "s_branch") or i + 1 == len(self.ins) else [i + 1]
            if x.op.startswith(("s_branch", "s_cbranch")):
                go.append(at[x.line.split(" ")[1]])
            assert not x.op.startswith(("s_setpc", "s_swappc"))
            self.succ.append(go)
        self.pred = [[] for _ in self.ins]
        for i, go in enumerate(self.succ):
            for j in go:
                self.pred[j].append(i)

    def near(self, i, edges, states):
        """Instructions with fewer than `states` wait states between them and instruction i, along any path."""
        best, todo = {}, [(j, states) for j in edges[i]]
        while todo:
            j, left = todo.pop()
            if left <= 0 or best.get(j, 0) >= left:
                continue
            best[j] = left
            todo += [(k, left - self.ins[j].states) for k in edges[j]]
        return best

    def hazards(self):
        found = []
        for i, x in enumerate(self.ins):
            if not x.mfma:
                continue
            for j in self.near(i, self.pred, BEFORE):
                y = self.ins[j]
                if y.vector and not y.mfma and y.writes & x.reads:
                    found.append(y.line + "  ->  " + x.line)
            for j in self.near(i, self.succ, AFTER):
                y = self.ins[j]
                # an MFMA that accumulates into the same registers is held back by the hardware
                touched = y.reads | y.writes if not y.mfma else y.reads | y.writes if x.writes != y.writes else set()
                if touched & x.writes:
                    found.append(x.line + "  ->  " + y.line)
        return found


def compiled(source, kernel, tmp_path):
    flags = [f for f in b.FLAGS if f != "-shared"]
    r = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--cuda-device-only", "-S",
                        "-Rpass-analysis=kernel-resource-usage", os.path.join(b.CSRC, source), "-o", str(tmp_path / "k.s")],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    mine = [u for u in r.stdout.split("Function Name: ") if kernel in u.splitlines()[0]]
    assert len(mine) == 1
    return mine[0], (tmp_path / "k.s").read_text()


@pytest.mark.parametrize("source,kernel,mfmas,exps,turns", [("attn_pipe.hip", "attn_pipe_kernel", 64, 32, 8),
                                                            ("attn_duo.hip", "attn_duo_kernel", 32, 16, 10),
                                                            ("attn_duo.hip", "attn_duo_suffix_kernel", 32, 16, 10)])
def test_no_register_is_spilled(source, kernel, mfmas, exps, turns, tmp_path):
    usage, asm = compiled(source, kernel, tmp_path)
    assert re.search(r"VGPRs Spill: 0\b", usage) and re.search(r"ScratchSize \[bytes/lane\]: 0\b", usage), usage
    # the steady loop: no move between architectural and accumulation registers among its MFMAs
    steady = [x for x in re.split(r"^\.LBB\w+:", asm, flags=re.M) if x.count("v_mfma") == mfmas and x.count("v_exp_f32") == exps]
    assert len(steady) >= turns
    assert all("v_accvgpr" not in x for x in steady)
    # everywhere: no vector instruction within the wait states of an MFMA's operands or result, along any branch
    code = Code(asm, kernel)
    assert sum(x.mfma for x in code.ins) >= turns * mfmas
    assert code.hazards() == []


def test_the_scan_finds_what_it_looks_for():
    def scan(*lines):
        return len(Code("k_fn:\n" + "".join("\t%s\n" % x if not x.endswith(":") else x + "\n" for x in lines) + ".Lfunc_end0:\n", "k_fn").hazards())
    m = "v_mfma_f32_16x16x32_bf16 v[0:3], v[8:11], v[12:15], v[0:3]"
    assert scan(m, m, "s_nop 10", "v_add_f32_e32 v4, v0, v1", "s_endpgm") == 0
    assert scan(m, "s_nop 9", "v_add_f32_e32 v4, v0, v5", "s_endpgm") == 1               # result read too early
    assert scan(m, "s_nop 9", "global_store_dwordx4 v[20:21], v[0:3], off", "s_endpgm") == 1
    assert scan(m, "s_cbranch_scc1 .LBB0_1", "s_nop 15", "s_endpgm", ".LBB0_1:", "v_mov_b32_e32 v2, 0", "s_endpgm") == 1
    assert scan("v_mov_b32_e32 v8, v30", "s_nop 1", m, "s_endpgm") == 0
    assert scan("v_mov_b32_e32 v8, v30", "s_nop 0", m, "s_endpgm") == 1                   # operand written too late
    assert scan("v_mov_b32_e32 v13, v30", "s_branch .LBB0_1", "s_nop 7", ".LBB0_1:", m, "s_endpgm") == 1
    assert scan("v_accvgpr_write_b32 a1, v30", "v_mfma_f32_16x16x32_bf16 a[0:3], v[8:11], v[12:15], a[0:3]", "s_endpgm") == 1
    assert scan("ds_read_b128 v[8:11], v40", "s_waitcnt lgkmcnt(0)", m, "s_endpgm") == 0
