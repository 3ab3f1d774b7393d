"""Host-side planning of the packed-rows kernel: which tiling, how many pieces.  Compiles attn_plan.cpp with a small driver
(no GPU)."""
import os
import subprocess

import pytest

from paper_2603_21257_amd import build as b

DRIVER = r"""
#include <cstdio>

#include "attn_plan.h"

namespace calvo {
int attn_pipe_tile_tokens(int heads_per_wg) { return 64 * (4 / heads_per_wg); }
int attn_duo_tile_tokens(int heads_per_wg) { return 32 * (4 / heads_per_wg); }
}
using namespace calvo;

// a line "f32 head_dim q_heads kv_heads cus forced_pieces room n, n times prefix suffix" -> "rows pieces items slots"
int main() {
  int f32, dim, hq, hkv, cus, force, room, n;
  while (scanf("%d %d %d %d %d %d %d %d", &f32, &dim, &hq, &hkv, &cus, &force, &room, &n) == 8) {
    std::vector<int32_t> blocks(n), suffix(n);
    for (int i = 0; i < n; i++) {
      if (scanf("%d %d", &blocks[i], &suffix[i]) != 2) return 1;
      blocks[i] /= 16;
    }
    const RowsPlan p = plan_rows(f32, dim, blocks.data(), suffix.data(), n, hq / hkv, hkv, cus, force, room);
    const PlanItems it = plan_items(p.tiles, p.want, rows_plan_params(p.shape, hkv, cus, force));
    printf("%d %d %zu %zu\n", p.shape.tile_rows, p.want, it.items.size(),
           it.split_tiles.empty() ? (size_t)0 : it.items.size() * hkv * p.shape.slots);
  }
}
"""


def compiled(tmp, source):
    (tmp / "driver.cpp").write_text(source)
    exe = tmp / "driver"
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", b.CSRC, str(tmp / "driver.cpp"), os.path.join(b.CSRC, "attn_plan.cpp"), "-o", str(exe)],
                   check=True)
    return exe


@pytest.fixture(scope="module")
def rows_plan(tmp_path_factory):
    exe = compiled(tmp_path_factory.mktemp("rows"), DRIVER)

    def ask(dtype, dim, hq, hkv, lens, cus=256, force=0, room=4096):
        line = [int(dtype == "f32"), dim, hq, hkv, cus, force, room, len(lens)] + [x for ps in lens for x in ps]
        out = subprocess.run([str(exe)], input=" ".join(map(str, line)), check=True, capture_output=True, text=True).stdout.split()
        return dict(zip(("rows", "pieces", "items", "slots"), map(int, out)))
    return ask


SMALL = {("bf16", 64): 32, ("bf16", 120): 32, ("bf16", 200): 16, ("bf16", 256): 16, ("f32", 256): 16}


@pytest.mark.parametrize("dtype,dim,hq,hkv,lens", [
    ("bf16", 256, 6, 3, [(256, 150)]), ("bf16", 200, 32, 8, [(432, 31)]), ("bf16", 256, 8, 8, [(400, 78)]),
    ("bf16", 256, 16, 1, [(384, 39)]), ("bf16", 120, 16, 4, [(0, 515)]), ("bf16", 256, 10, 2, [(304, 120)])])
def test_a_longer_launch_is_not_taken_for_less_load(rows_plan, dtype, dim, hq, hkv, lens):
    """Few tiles over a short context: cut in the smaller tiling, or of it, the launch is a fifth shorter."""
    assert rows_plan(dtype, dim, hq, hkv, lens)["rows"] == SMALL[dtype, dim]
