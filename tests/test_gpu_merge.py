"""The kernel that merges split-KV pieces, at the piece counts where its batches end: around one batch of
eight loads, around one wave of 64 pieces, and far beyond it (a layer loaded in two-block chunks)."""
import pytest

import hip_harness as hh
from paper_2603_21257_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pieces", [2, 7, 8, 9, 63, 64])
def test_forced_piece_counts(pieces, monkeypatch):
    monkeypatch.setenv("CALVO_ATTN_SPLITS", str(pieces))
    w = wl.make_custom(wl.Shape(1, 8, 2, 128, "bf16", 200), [(2560, 33), (64, 5)], seed=600 + pieces)
    print(f"[case] pieces={pieces}", flush=True)
    pool_g, out_g = hh.run_hip(w)
    pool_o, out_o = hh.run_oracle(w)
    hh.assert_pool_bit_exact(pool_g, pool_o)
    hh.assert_attn_close(out_g, out_o, "bf16")


@pytest.mark.parametrize("prefix_blocks", [126, 128, 130, 261])
def test_more_pieces_than_lanes(prefix_blocks):
    """One piece per two-block chunk and one for the rest: 64, 65, 66 and 131 pieces (63 to 130 chunks)."""
    w = wl.make_custom(wl.Shape(1, 10, 2, 128, "bf16", 280), [(16 * prefix_blocks, 21)], seed=700 + prefix_blocks)
    print(f"[case] prefix_blocks={prefix_blocks}", flush=True)
    pool_g, out_g = hh.run_hip(w, chunk_blocks=[2])
    pool_o, out_o = hh.run_oracle(w)
    hh.assert_pool_bit_exact(pool_g, pool_o)
    hh.assert_attn_close(out_g, out_o, "bf16")
