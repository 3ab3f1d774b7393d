"""The packed-rows attention kernel (fp32 pools, head widths other than 128) where its tiling can go wrong:
head widths around its padded widths, groups that do not divide a 16-row block, row counts around a wave and
a workgroup, contexts around a step, cut contexts, several requests, tokens that later rows must not see."""
import numpy as np
import pytest
import torch

import hip_harness as hh
from paper_2603_21257_amd import binding as cb
from paper_2603_21257_amd import workload as wl

pytestmark = pytest.mark.gpu


def check(w, **kw):
    print(f"[case] shape={w.shape} lens={[(r.prefix_len, r.suffix_len) for r in w.requests]} kw={kw}", flush=True)
    pool_g, out_g = hh.run_hip(w, **kw)
    pool_o, out_o = hh.run_oracle(w, scale=kw.get("scale") or None)
    if kw.get("append_suffix", True):
        hh.assert_pool_bit_exact(pool_g, pool_o)
    hh.assert_attn_close(out_g, out_o, w.shape.dtype)


def slots(lens):
    return sum(-(-(p + s) // 16) for p, s in lens) + 8


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D", [8, 40, 64, 72, 96, 136, 200, 256])
def test_head_widths(dtype, D):
    lens = [(96, 70)]
    check(wl.make_custom(wl.Shape(1, 6, 2, D, dtype, slots(lens)), lens, seed=D))


def test_head_width_128_fp32():
    lens = [(160, 37)]
    check(wl.make_custom(wl.Shape(1, 8, 2, 128, "f32", slots(lens)), lens, seed=128))


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("bf16", 64), ("bf16", 256)])
@pytest.mark.parametrize("hq,hkv", [(1, 1), (5, 1), (10, 2), (16, 8), (34, 2)])
@pytest.mark.parametrize("P,S", [(0, 1), (0, 17), (16, 1), (32, 15), (48, 33), (496, 5)])
def test_groups_and_edges(dtype, D, hq, hkv, P, S):
    check(wl.make_custom(wl.Shape(1, hq, hkv, D, dtype, slots([(P, S)])), [(P, S)], seed=hq + P + S))


@pytest.mark.parametrize("pieces", [0, 2, 7, 64])
@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f32", 128), ("f32", 256), ("bf16", 96), ("bf16", 256)])
def test_cut_contexts(dtype, D, pieces, monkeypatch):
    if pieces:
        monkeypatch.setenv("CALVO_ATTN_SPLITS", str(pieces))
    lens = [(2064, 19)]
    check(wl.make_custom(wl.Shape(1, 6, 2, D, dtype, slots(lens)), lens, seed=pieces + D))


@pytest.mark.parametrize("pieces", [0, 3])
@pytest.mark.parametrize("D,hq,hkv", [(-136, 6, 2), (-256, 10, 2), (8, 1, 1), (40, 6, 2), (64, 8, 2), (64, 34, 2), (72, 5, 1), (120, 6, 2), (136, 6, 2), (256, 8, 8), (256, 10, 2)])
@pytest.mark.parametrize("lens", [[(0, 1)], [(16, 7)], [(32, 15), (496, 33)], [(2064, 130), (0, 64), (48, 1)]])
def test_large_tiling(D, hq, hkv, lens, pieces, monkeypatch):
    """The tiling of twice the rows, which short suffixes get in no other way: rows around a tile, one step and many per wave.
    Head widths below 0: fp32."""
    monkeypatch.setenv("CALVO_ROWS_TILE", "2")
    if pieces:
        monkeypatch.setenv("CALVO_ATTN_SPLITS", str(pieces))
    rows = []
    check(wl.make_custom(wl.Shape(1, hq, hkv, abs(D), "f32" if D < 0 else "bf16", slots(lens)), lens, seed=abs(D) + hq + pieces),
          look=lambda ctx: rows.append(cb.calvo_attn_tile_rows(ctx, 0)))
    assert rows == [64 if 0 < D <= 128 else 32]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_many_rows_several_requests(dtype):
    """Enough tiles for several rounds of workgroups, next to tiny requests."""
    lens = [(64, 700), (0, 1), (320, 515), (16, 0), (1600, 3)]
    w = wl.make_custom(wl.Shape(1, 64, 16, 64, dtype, slots(lens)), lens, seed=11)
    check(w)
    check(wl.make_custom(wl.Shape(2, 8, 2, 64, dtype, 400), [(640, 90), (512, 33)], seed=12, shared_blocks=20), prepared=True)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("fn", [cb.calvo_prefill_attn, cb.calvo_prefill_attn_noalloc])
def test_entry_points(dtype, fn):
    lens = [(1024, 45)]
    check(wl.make_custom(wl.Shape(2, 8, 2, 80, dtype, slots(lens)), lens, seed=21), attn_fn=fn, scale=0.2)


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f32", 256), ("bf16", 64), ("bf16", 256)])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("tile", ["1", "2"])
def test_later_tokens_do_not_reach_earlier_rows(dtype, D, value, tile, monkeypatch):
    """V of token 20 is not finite: rows 0..19 are what the oracle gives for finite values (their keys are walked again
    one by one, a different order of the same sums), rows from 20 on what it gives for this one."""
    monkeypatch.setenv("CALVO_ROWS_TILE", tile)
    w = wl.make_custom(wl.Shape(1, 6, 2, D, dtype, 32), [(64, 40)], seed=31)
    _, want = hh.run_oracle(w)
    bad = np.float32(value).view(np.uint32)
    w.v_suffix[0, 20] = np.uint16(bad >> 16) if dtype == "bf16" else np.float32(value)
    _, got = hh.run_hip(w)
    hh.assert_attn_close(got[:, :20], want[:, :20], dtype)
    wide = hh.orc.widen(got) if dtype == "bf16" else got
    with np.errstate(invalid="ignore"):
        _, want = hh.run_oracle(w)
    assert np.array_equal(wide[0, 20:], want[0, 20:], equal_nan=True)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_prefix_that_another_request_of_the_call_appends(dtype):
    """One sequence as two requests: the second one's cached prefix is what the first one appends."""
    s = wl.Shape(1, 8, 2, 64, dtype, 64)
    w = wl.make_custom(s, [(0, 64), (64, 30)], seed=41)
    first, second = w.requests
    table = second.table.copy()
    table[:4] = first.table[:4]
    dev, dt = torch.device("cuda:0"), hh.torch_dtype(s)
    pool = hh.to_torch(hh.sentinel_pool_np(s), s, dev)
    q, ks, vs = (hh.to_torch(a, s, dev) for a in (w.q, w.k_suffix, w.v_suffix))
    out = torch.empty((w.total_suffix, s.n_q_heads, s.head_dim), dtype=dt, device=dev)
    torch.cuda.synchronize()
    ctx = cb.calvo_create(1, s.n_q_heads, s.n_kv_heads, s.head_dim, cb.CALVO_BF16 if dtype == "bf16" else cb.CALVO_F32, s.pool_blocks, pool)
    try:
        reqs = [cb.make_request(None, 0, first.table, 0, 64), cb.make_request(None, 0, table, 4, 30, 4)]
        cb.calvo_prefill_attn(ctx, 0, q[0], ks[0], vs[0], out, reqs, w.cu_suffix)
    finally:
        cb.calvo_destroy(ctx)
    torch.cuda.synchronize()
    # the oracle sees the same as one request of 94 tokens
    one = wl.make_custom(s, [(0, 94)], seed=42)
    one.q, one.k_suffix, one.v_suffix = w.q, w.k_suffix, w.v_suffix
    _, want = hh.run_oracle(one)
    hh.assert_attn_close(hh.to_numpy_stored(out[None], s), want, dtype)
