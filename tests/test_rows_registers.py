"""The compiled packed-rows kernels (no GPU needed): no scratch memory, and the loads that the merge has in flight."""
import os
import re
import subprocess

import pytest

from paper_2603_21257_amd import build as b


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = tmp_path_factory.mktemp("rows") / "k.s"
    flags = [f for f in b.FLAGS if f != "-shared"]
    r = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--cuda-device-only", "-S", os.path.join(b.CSRC, "attn_rows.hip"),
                        "-o", str(out)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    return out.read_text()


@pytest.fixture(scope="module")
def compiled(assembly):
    """By mangled kernel name."""
    return dict(re.findall(r"^(_ZN5calvo4rows\w+):[^\n]*\n(.*?)^\.Lfunc_end", assembly, re.M | re.S))


@pytest.mark.parametrize("dim,load", [(64, "global_load_dword "), (128, "global_load_dwordx2 "), (256, "global_load_dwordx4 ")])
def test_merge_has_eight_pieces_in_flight(compiled, dim, load):
    """Twice: in front of the weights, and in the loop over what is left."""
    merges = {k: v for k, v in compiled.items() if re.search(r"merge_rows_kernelI[ft]Li%dE" % dim, k)}
    assert len(merges) >= 2
    for name, asm in merges.items():
        assert len(re.findall(load, re.sub(r"[ \t]+", " ", asm))) >= 16, name


def test_no_scratch_memory(assembly):
    """The widest partly filled heads in the larger tiling put two registers aside, into accumulation registers."""
    spills = {}
    for entry in re.split(r"^  - \.agpr_count:", assembly, flags=re.M)[1:]:
        name = re.search(r"\.name: +(\S+)", entry).group(1)
        assert re.search(r"\.private_segment_fixed_size: 0\n", entry), name
        n = int(re.search(r"\.vgpr_spill_count: (\d+)", entry).group(1))
        if "rows_kernel" in name:
            spills[name] = n
    assert len([k for k in spills if "attn_rows_kernel" in k]) == 18
    assert all(n <= (2 if "RowsCfgItLi128ELi4ELi2ELi4ELb0E" in k else 0) for k, n in spills.items()), spills
