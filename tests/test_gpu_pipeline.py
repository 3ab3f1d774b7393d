"""Both shapes of the attention kernel (64 and 32 query rows per wave) at the lengths where its loops change: number of whole sub-tiles in front of the diagonal
around fill, one pair of steps, one turn of the ring and what is left behind them; one to nine sub-tiles on the diagonal
(groups of one head take 256 tokens per tile, requested in two groups); empty row blocks; cut contexts; a key that
raises the softmax reference in every position of a turn."""
import numpy as np
import pytest

import hip_harness as hh
from paper_2603_21257_amd import workload as wl

pytestmark = pytest.mark.gpu


def check(w):
    print(f"[case] shape={w.shape} lens={[(r.prefix_len, r.suffix_len) for r in w.requests]}", flush=True)
    pool_g, out_g = hh.run_hip(w)
    pool_o, out_o = hh.run_oracle(w)
    hh.assert_pool_bit_exact(pool_g, pool_o)
    hh.assert_attn_close(out_g, out_o, "bf16")


@pytest.mark.parametrize("subs", [0, 1, 2, 3, 4, 5, 8, 9, 10, 11, 12, 13, 17, 18, 22, 26, 27])
@pytest.mark.parametrize("half", [0, 16])
@pytest.mark.parametrize("variant", ["3", "4"])
def test_whole_sub_tiles_in_front_of_the_diagonal(subs, half, variant, monkeypatch):
    monkeypatch.setenv("CALVO_ATTN_VARIANT", variant)
    P = 32 * subs + half
    check(wl.make_custom(wl.Shape(1, 8, 2, 128, "bf16", (P + 64) // 16 + 9), [(P, 64 - half // 2)], seed=800 + subs + half))


@pytest.mark.parametrize("hq,hkv,S", [(3, 1, 300), (3, 1, 256), (10, 5, 130), (8, 2, 33), (8, 2, 70), (6, 1, 128), (2, 2, 511)])
@pytest.mark.parametrize("pieces", [0, 2, 5])
@pytest.mark.parametrize("variant", ["3", "4"])
def test_row_blocks_and_pieces(hq, hkv, S, pieces, variant, monkeypatch):
    monkeypatch.setenv("CALVO_ATTN_VARIANT", variant)
    if pieces:
        monkeypatch.setenv("CALVO_ATTN_SPLITS", str(pieces))
    check(wl.make_custom(wl.Shape(1, hq, hkv, 128, "bf16", (1200 + 2 * S) // 16 + 40), [(656, S), (272, S // 2)], seed=830 + S))


@pytest.mark.parametrize("sub", list(range(1, 25)))
@pytest.mark.parametrize("variant", ["3", "4"])
def test_reference_raised_anywhere_in_a_turn(sub, variant, monkeypatch):
    """One key of sub-tile `sub` is 120 times as long as the others: its scores pass the reference by far more than 2^16."""
    monkeypatch.setenv("CALVO_ATTN_VARIANT", variant)
    P, S = 32 * 25, 64
    s = wl.Shape(1, 4, 1, 128, "bf16", (P + S) // 16 + 5)
    w = wl.make_custom(s, [(P, S)], seed=870 + sub)
    host = w.host_kv.reshape(1, -1, 2, 16, s.n_kv_heads, s.head_dim)
    pos = 32 * sub + 7 * sub % 32
    b, t = w.requests[0].host_block_start + pos // 16, pos % 16
    import torch
    row = torch.from_numpy(host[0, b, 0, t].view(np.int16).copy()).view(torch.bfloat16) * 120
    host[0, b, 0, t] = row.view(torch.int16).numpy().view(np.uint16)
    check(w)


@pytest.mark.parametrize("variant", ["3", "4"])
@pytest.mark.parametrize("pieces", [7, 15])
def test_blocks_that_come_from_memory(variant, pieces, monkeypatch):
    """Every layer is read for the first time, right behind its load: requests take longest, a wait that counts one too few
    shows in the first steps of a piece."""
    monkeypatch.setenv("CALVO_ATTN_VARIANT", variant)
    monkeypatch.setenv("CALVO_ATTN_SPLITS", str(pieces))
    lens = [(4096, 3), (8192, 70), (6144, 130)]
    check(wl.make_custom(wl.Shape(3, 8, 2, 128, "bf16", 1250), lens, seed=900 + pieces))
