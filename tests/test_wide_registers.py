"""The long-suffix attention kernel writes its MFMAs as inline assembly and keeps every value in a register of its own: with
a single spilled or moved operand the wait states that it counts on are gone.  Compiles the kernel (no GPU needed)."""
import os
import re
import subprocess

from paper_2603_21257_amd import build as b


def test_no_register_is_spilled(tmp_path):
    flags = [f for f in b.FLAGS if f != "-shared"]
    r = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--cuda-device-only", "-S",
                        "-Rpass-analysis=kernel-resource-usage", os.path.join(b.CSRC, "attn_pipe.hip"), "-o", str(tmp_path / "k.s")],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    usage = r.stdout.split("Function Name: ")
    mine = [u for u in usage if "attn_pipe_kernel" in u.splitlines()[0]]
    assert len(mine) == 1
    assert re.search(r"VGPRs Spill: 0\b", mine[0]) and re.search(r"ScratchSize \[bytes/lane\]: 0\b", mine[0]), mine[0]
    # the steady loop: no move between architectural and accumulation registers among its MFMAs
    asm = (tmp_path / "k.s").read_text()
    blocks = re.split(r"^\.LBB\w+:", asm, flags=re.M)
    steady = [x for x in blocks if x.count("v_mfma") == 64 and x.count("v_exp_f32") == 32]
    assert len(steady) >= 8
    assert all("v_accvgpr" not in x for x in steady)
