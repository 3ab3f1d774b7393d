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

// a line "f32 head_dim q_heads kv_heads cus forced_pieces forced_tiling room n, n times prefix suffix" -> "rows pieces items slots"
int main() {
  int f32, dim, hq, hkv, cus, force, tile, room, n;
  while (scanf("%d %d %d %d %d %d %d %d %d", &f32, &dim, &hq, &hkv, &cus, &force, &tile, &room, &n) == 9) {
    std::vector<int32_t> blocks(n), suffix(n);
    for (int i = 0; i < n; i++) {
      if (scanf("%d %d", &blocks[i], &suffix[i]) != 2) return 1;
      blocks[i] /= 16;
    }
    const RowsPlan p = plan_rows(f32, dim, blocks.data(), suffix.data(), n, hq / hkv, hkv, cus, force, room, tile);
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

    def ask(dtype, dim, hq, hkv, lens, cus=256, force=0, tile=0, room=4096):
        line = [int(dtype == "f32"), dim, hq, hkv, cus, force, tile, room, len(lens)] + [x for ps in lens for x in ps]
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


@pytest.mark.parametrize("dtype,dim,hq,hkv,lens,rows", [
    ("bf16", 64, 32, 8, [(2048, 256)], 32), ("bf16", 64, 32, 8, [(8192, 512)], 64), ("bf16", 64, 32, 8, [(0, 512)], 64),
    ("bf16", 64, 16, 4, [(4096, 300)], 32), ("bf16", 96, 32, 8, [(8192, 128)], 64), ("bf16", 96, 8, 8, [(512, 400)], 32),
    ("bf16", 256, 32, 8, [(2048, 256)], 32), ("bf16", 256, 8, 2, [(2048, 16)], 16), ("f32", 256, 32, 8, [(2048, 256)], 32),
    ("f32", 256, 8, 2, [(1024, 60)], 16), ("f32", 128, 32, 8, [(8192, 512)], 32), ("f32", 64, 32, 8, [(8192, 512)], 32),
    ("bf16", 200, 40, 8, [(240, 386), (8720, 63), (2224, 3)], 32)])            # a longer launch on a full chip
def test_which_tiling(rows_plan, dtype, dim, hq, hkv, lens, rows):
    assert rows_plan(dtype, dim, hq, hkv, lens)["rows"] == rows


@pytest.mark.parametrize("dtype,dim", [("bf16", 40), ("bf16", 96), ("bf16", 256), ("f32", 64), ("f32", 256)])
@pytest.mark.parametrize("room", [64, 512, 4096])
def test_pieces_fit_the_room_for_partial_results(rows_plan, dtype, dim, room):
    """A slot is 32 rows of 128 floats: 64 rows, or 32 of 256-wide heads, take two."""
    for lens in [(512, 1)], [(8192, 20)], [(2048, 256)], [(32768, 64)], [(8192, 128), (4096, 3), (0, 70)]:
        for hq, hkv in (8, 2), (32, 8):
            p = rows_plan(dtype, dim, hq, hkv, lens, room=room)
            assert p["slots"] <= room
            rows = max(p["rows"] * (64 if dim <= 64 else 128 if dim <= 128 else 256) // 128, p["rows"]) / 32
            assert p["slots"] % p["items"] == 0 and (p["slots"] == 0 or p["slots"] // p["items"] >= hkv * rows)


def test_a_decision_that_fails_is_not_kept(tmp_path):
    """Host memory that runs out while a batch is planned: the next call with its lengths decides again."""
    exe = compiled(tmp_path, DRIVER.split("// a line")[0] + r"""
#include <new>

int main() {
  KeptPlan k;
  const int32_t a[] = {4, 2}, b[] = {8, 2};
  int made = 0;
  auto seven = [&](KeptPlan& p) { made++; p.want = 7; };
  auto fails = [&](KeptPlan&) { throw std::bad_alloc(); };
  if (k.of(3, a, a, 2, seven).want != 7 || k.of(3, a, a, 2, fails).want != 7 || made != 1) return 1;
  try { k.of(3, b, a, 2, fails); return 2; } catch (const std::bad_alloc&) {}
  k.of(3, b, a, 2, [&](KeptPlan& p) { made++; p.want = 9; });
  if (made != 2 || k.want != 9) return 3;
  k.of(4, b, a, 2, seven);          // another kernel
  k.of(4, b, a, 1, seven);          // fewer requests
  return made == 4 ? 0 : 4;
}
""")
    assert subprocess.run([str(exe)]).returncode == 0


@pytest.mark.parametrize("force", [0, 3])
@pytest.mark.parametrize("dtype,dim,sizes", [("bf16", 64, (32, 64)), ("bf16", 96, (32, 64)), ("bf16", 256, (16, 32)), ("f32", 64, (32, 32)),
                                             ("f32", 128, (32, 32)), ("f32", 136, (16, 32))])
def test_a_forced_tiling(rows_plan, dtype, dim, sizes, force):
    for lens in [(64, 1)], [(8192, 512)], [(2064, 130), (0, 64), (48, 1)]:
        assert tuple(rows_plan(dtype, dim, 8, 2, lens, tile=t, force=force)["rows"] for t in (1, 2)) == sizes
