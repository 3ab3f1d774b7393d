"""A suffix of one tile: the pipelined kernels read its rows from the caller's arrays and store them to the pool
themselves.  Lengths around a block, a 32-key sub-tile and the tile; odd and even prefix block counts (the first suffix
block shares a sub-tile with the prefix or not); groups with one, two and several head groups per KV head; cut contexts;
both workgroup shapes; without suffix arrays the pool's rows are used."""
import pytest
import torch

import hip_harness as hh
from paper_2603_21257_amd import binding as cb
from paper_2603_21257_amd import workload as wl

pytestmark = pytest.mark.gpu


def check(shape, lens, seed, **kw):
    w = wl.make_custom(shape, lens, seed=seed)
    print(f"[case] shape={w.shape} lens={lens} kw={kw}", flush=True)
    pool_g, out_g = hh.run_hip(w, **kw)
    pool_o, out_o = hh.run_oracle(w)
    hh.assert_pool_bit_exact(pool_g, pool_o)
    hh.assert_attn_close(out_g, out_o, "bf16")


@pytest.mark.parametrize("variant", [0, 3, 4])
@pytest.mark.parametrize("P", [0, 16, 32, 48, 272, 1040])
@pytest.mark.parametrize("S", [1, 15, 16, 17, 31, 32, 33, 64, 65])
def test_around_the_tile(variant, P, S, monkeypatch):
    if variant:
        monkeypatch.setenv("CALVO_ATTN_VARIANT", str(variant))
    check(wl.Shape(1, 8, 2, 128, "bf16", (P + S) // 16 + 9), [(P, S)], seed=P + S)


@pytest.mark.parametrize("hq,hkv,S", [(16, 2, 20), (5, 1, 100), (5, 1, 129), (10, 2, 255), (12, 2, 50), (2, 2, 128), (32, 8, 9)])
@pytest.mark.parametrize("pieces", [0, 3])
def test_head_groups_and_pieces(hq, hkv, S, pieces, monkeypatch):
    if pieces:
        monkeypatch.setenv("CALVO_ATTN_SPLITS", str(pieces))
    P = 2064
    check(wl.Shape(2, hq, hkv, 128, "bf16", (P + S) // 16 + 9), [(P, S)], seed=hq + S)


@pytest.mark.parametrize("kw", [dict(prepared=True), dict(attn_fn=cb.calvo_prefill_attn_noalloc), dict(chunk_blocks=[20]), dict(staging_bytes=1 << 20)])
def test_entry_points(kw):
    check(wl.Shape(1, 8, 2, 128, "bf16", 120), [(1552, 27)], seed=9, **kw)


@pytest.mark.parametrize("dtype,D,heads,P,S", [("f32", 64, 4, 96, 300), ("bf16", 96, 8, 96, 300), ("bf16", 128, 4, 2064, 25),
                                              ("bf16", 128, 1, 48, 128), ("bf16", 128, 4, 96, 300)])
@pytest.mark.parametrize("over", ["k", "v"])
def test_output_over_the_suffix_rows(dtype, D, heads, P, S, over):
    """As many KV heads as query heads and the output in the place of k_suffix or v_suffix: the rows are read first."""
    s = wl.Shape(1, heads, heads, D, dtype, (P + S) // 16 + 9)
    w = wl.make_custom(s, [(P, S)], seed=960 + S)
    dev = torch.device("cuda:0")
    pool = hh.to_torch(hh.sentinel_pool_np(s), s, dev)
    host = hh.to_torch(w.host_kv, s, pin=True)
    q, ks, vs = (hh.to_torch(a, s, dev) for a in (w.q, w.k_suffix, w.v_suffix))
    out = ks if over == "k" else vs
    torch.cuda.synchronize()
    ctx = cb.calvo_create(1, heads, heads, D, cb.CALVO_BF16 if dtype == "bf16" else cb.CALVO_F32, s.pool_blocks, pool)
    try:
        reqs = hh.make_requests(w, host)
        cb.calvo_kv_ingest(ctx, reqs, 0, 1)
        cb.calvo_prefill_attn(ctx, 0, q[0], ks[0], vs[0], out[0], reqs, w.cu_suffix)
    finally:
        cb.calvo_destroy(ctx)
    torch.cuda.synchronize()
    pool_o, want = hh.run_oracle(w)
    hh.assert_pool_bit_exact(hh.to_numpy_stored(pool, s), pool_o)
    hh.assert_attn_close(hh.to_numpy_stored(out, s), want, dtype)
