"""The pipelined attention kernels write their MFMAs as inline assembly and keep every value in a register of its own: with
a single spilled or moved operand the wait states that they count on are gone.  Compiles the kernels (no GPU needed)."""
import os
import re
import subprocess

import pytest

from paper_2603_21257_amd import build as b


@pytest.mark.parametrize("source,kernel,mfmas,exps,turns", [("attn_pipe.hip", "attn_pipe_kernel", 64, 32, 8),
                                                            ("attn_duo.hip", "attn_duo_kernel", 32, 16, 10)])
def test_no_register_is_spilled(source, kernel, mfmas, exps, turns, tmp_path):
    flags = [f for f in b.FLAGS if f != "-shared"]
    r = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--cuda-device-only", "-S",
                        "-Rpass-analysis=kernel-resource-usage", os.path.join(b.CSRC, source), "-o", str(tmp_path / "k.s")],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    mine = [u for u in r.stdout.split("Function Name: ") if kernel in u.splitlines()[0]]
    assert len(mine) == 1
    assert re.search(r"VGPRs Spill: 0\b", mine[0]) and re.search(r"ScratchSize \[bytes/lane\]: 0\b", mine[0]), mine[0]
    # the steady loop: no move between architectural and accumulation registers among its MFMAs
    asm = (tmp_path / "k.s").read_text()
    steady = [x for x in re.split(r"^\.LBB\w+:", asm, flags=re.M) if x.count("v_mfma") == mfmas and x.count("v_exp_f32") == exps]
    assert len(steady) >= turns
    assert all("v_accvgpr" not in x for x in steady)
