"""The compiled packed-rows kernels (no GPU needed): loads that the merge has in flight."""
import os
import re
import subprocess

import pytest

from paper_2603_21257_amd import build as b


@pytest.fixture(scope="module")
def compiled(tmp_path_factory):
    """Assembly by mangled kernel name."""
    out = tmp_path_factory.mktemp("rows") / "k.s"
    flags = [f for f in b.FLAGS if f != "-shared"]
    r = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--cuda-device-only", "-S", os.path.join(b.CSRC, "attn_rows.hip"),
                        "-o", str(out)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    return dict(re.findall(r"^(_ZN5calvo4rows\w+):[^\n]*\n(.*?)^\.Lfunc_end", out.read_text(), re.M | re.S))


@pytest.mark.parametrize("dim,load", [(64, "global_load_dword "), (128, "global_load_dwordx2 "), (256, "global_load_dwordx4 ")])
def test_merge_has_eight_pieces_in_flight(compiled, dim, load):
    """Twice: in front of the weights, and in the loop over what is left."""
    merges = {k: v for k, v in compiled.items() if re.search(r"merge_rows_kernelI[ft]Li%dE" % dim, k)}
    assert len(merges) >= 2
    for name, asm in merges.items():
        assert len(re.findall(load, re.sub(r"[ \t]+", " ", asm))) >= 16, name
