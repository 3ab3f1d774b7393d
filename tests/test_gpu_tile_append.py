"""Suffixes whose rows the pipelined kernels read from the caller's arrays and store to the pool themselves: one tile, and in
small tiles any length, also of several requests.  Lengths around a block, a 32-key sub-tile, the tile and 400 tokens; odd
and even prefix block counts (the first suffix block shares a sub-tile with the prefix or not); groups with one, two and several
head groups per KV head; cut contexts; both workgroup shapes; without suffix arrays the pool's rows are used."""
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


@pytest.mark.parametrize("heads", [(8, 2), (5, 1), (32, 8)])
@pytest.mark.parametrize("P,S", [(0, 200), (16, 97), (48, 161), (336, 399), (320, 400), (336, 401), (1040, 260)])
@pytest.mark.parametrize("pieces", [0, 2, 5])
def test_several_tiles(heads, P, S, pieces, monkeypatch):
    monkeypatch.setenv("CALVO_ATTN_VARIANT", "4")
    if pieces:
        monkeypatch.setenv("CALVO_ATTN_SPLITS", str(pieces))
    check(wl.Shape(1, *heads, 128, "bf16", (P + S) // 16 + 9), [(P, S)], seed=P + S + pieces)


@pytest.mark.parametrize("heads", [(8, 2), (5, 1), (16, 8)])
@pytest.mark.parametrize("lens", [[(0, 1100)], [(448, 607)], [(1040, 700)], [(2064, 530)], [(0, 600), (528, 450), (64, 3)]])
@pytest.mark.parametrize("pieces", [0, 3])
def test_long_suffixes_in_small_tiles(heads, lens, pieces, monkeypatch):
    """Turns of the loop within the prefix, across its end and within the suffix."""
    monkeypatch.setenv("CALVO_ATTN_VARIANT", "4")
    if pieces:
        monkeypatch.setenv("CALVO_ATTN_SPLITS", str(pieces))
    check(wl.Shape(1, *heads, 128, "bf16", sum((p + s) // 16 + 1 for p, s in lens) + 9), lens, seed=lens[0][1] + pieces)


@pytest.mark.parametrize("lens,shared", [([(64, 1), (0, 90), (272, 33), (16, 0)], 0), ([(160, 70), (112, 400), (96, 17)], 5), ([(48, 401), (48, 2)], 0)])
@pytest.mark.parametrize("prepared", [False, True])
def test_several_requests(lens, shared, prepared, monkeypatch):
    monkeypatch.setenv("CALVO_ATTN_VARIANT", "4")
    w = wl.make_custom(wl.Shape(2, 16, 2, 128, "bf16", 80), lens, seed=len(lens) + shared, shared_blocks=shared)
    print(f"[case] lens={lens} shared={shared}", flush=True)
    pool_g, out_g = hh.run_hip(w, prepared=prepared)
    pool_o, out_o = hh.run_oracle(w)
    hh.assert_pool_bit_exact(pool_g, pool_o)
    hh.assert_attn_close(out_g, out_o, "bf16")


@pytest.mark.parametrize("variant", ["3", "4"])
def test_prefix_that_another_request_of_the_call_appends(variant, monkeypatch):
    """One sequence as two requests: what the second one has cached is what the first one appends, so all rows are stored first."""
    monkeypatch.setenv("CALVO_ATTN_VARIANT", variant)
    s = wl.Shape(1, 8, 2, 128, "bf16", 64)
    w = wl.make_custom(s, [(0, 64), (64, 30)], seed=43)
    first, second = w.requests
    table = second.table.copy()
    table[:4] = first.table[:4]
    dev = torch.device("cuda:0")
    pool = hh.to_torch(hh.sentinel_pool_np(s), s, dev)
    q, ks, vs = (hh.to_torch(a, s, dev) for a in (w.q, w.k_suffix, w.v_suffix))
    out = torch.empty((1, w.total_suffix, s.n_q_heads, s.head_dim), dtype=torch.bfloat16, device=dev)
    torch.cuda.synchronize()
    ctx = cb.calvo_create(1, s.n_q_heads, s.n_kv_heads, s.head_dim, cb.CALVO_BF16, s.pool_blocks, pool)
    try:
        reqs = [cb.make_request(None, 0, first.table, 0, 64), cb.make_request(None, 0, table, 4, 30, 4)]
        cb.calvo_prefill_attn(ctx, 0, q[0], ks[0], vs[0], out[0], reqs, w.cu_suffix)
    finally:
        cb.calvo_destroy(ctx)
    torch.cuda.synchronize()
    one = wl.make_custom(s, [(0, 94)], seed=44)          # the oracle sees the same as one request of 94 tokens
    one.q, one.k_suffix, one.v_suffix = w.q, w.k_suffix, w.v_suffix
    _, want = hh.run_oracle(one)
    hh.assert_attn_close(hh.to_numpy_stored(out, s), want, "bf16")


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


KERNELS = [("bf16", 64, ""), ("f32", 64, ""), ("bf16", 256, ""), ("bf16", 128, "3"), ("bf16", 128, "4")]


@pytest.mark.parametrize("dtype,D,variant", KERNELS)
@pytest.mark.parametrize("P,S,at_home", [(48, 16, True), (64, 5, True), (320, 11, False), (336, 401, False)])
def test_suffix_rows_in_the_pool(dtype, D, variant, P, S, at_home, monkeypatch):
    """k_suffix and v_suffix are rows of the layer's pool: of blocks that no table names, or the very rows they go to.  All
    rows are stored first."""
    monkeypatch.setenv("CALVO_ATTN_VARIANT", variant)
    s = wl.Shape(1, 8, 2, D, dtype, (P + S) // 16 + 9)
    w = wl.make_custom(s, [(P, S)], seed=970 + S)
    dev = torch.device("cuda:0")
    spare = -(-S // 16) + 1
    pool = torch.zeros((s.pool_blocks + spare, 2, 16, 2, D), dtype=hh.torch_dtype(s), device=dev)
    pool[:s.pool_blocks] = hh.to_torch(hh.sentinel_pool_np(s), s, dev).view(-1, 2, 16, 2, D)
    host = hh.to_torch(w.host_kv, s, pin=True)
    q, ks, vs = (hh.to_torch(a, s, dev) for a in (w.q, w.k_suffix, w.v_suffix))
    if at_home:
        home = pool[int(w.requests[0].table[P // 16])]
        k_rows, v_rows = home[0, :S], home[1, :S]
    else:
        k_rows, v_rows = pool[s.pool_blocks:].view(2, -1, 2, D)[:, :S]
    k_rows.copy_(ks[0])
    v_rows.copy_(vs[0])
    out = torch.empty((1, S, 8, D), dtype=pool.dtype, device=dev)
    torch.cuda.synchronize()
    ctx = cb.calvo_create(1, 8, 2, D, cb.CALVO_BF16 if dtype == "bf16" else cb.CALVO_F32, s.pool_blocks + spare, pool)
    try:
        reqs = hh.make_requests(w, host)
        cb.calvo_kv_ingest(ctx, reqs, 0, 1)
        cb.calvo_prefill_attn(ctx, 0, q[0], k_rows, v_rows, out[0], reqs, w.cu_suffix)
    finally:
        cb.calvo_destroy(ctx)
    torch.cuda.synchronize()
    pool_o, want = hh.run_oracle(w)
    hh.assert_pool_bit_exact(hh.to_numpy_stored(pool[:s.pool_blocks].reshape(1, s.pool_blocks, -1), s), pool_o)
    hh.assert_attn_close(hh.to_numpy_stored(out, s), want, dtype)


@pytest.mark.parametrize("dtype,D,variant", KERNELS)
@pytest.mark.parametrize("P,S", [(0, 5), (48, 40), (64, 130)])
def test_two_requests_that_append_to_the_same_slots(dtype, D, variant, P, S, monkeypatch):
    """One sequence twice, the same rows to the same slots, under other queries."""
    monkeypatch.setenv("CALVO_ATTN_VARIANT", variant)
    s = wl.Shape(1, 8, 2, D, dtype, 2 * ((P + S) // 16 + 9))
    w = wl.make_custom(s, [(P, S), (P, S)], seed=990 + S)
    first, second = w.requests
    second.table[:] = first.table
    second.host_block_start = first.host_block_start
    w.k_suffix[:, S:] = w.k_suffix[:, :S]
    w.v_suffix[:, S:] = w.v_suffix[:, :S]
    pool_g, out_g = hh.run_hip(w)
    pool_o, out_o = hh.run_oracle(w)
    hh.assert_pool_bit_exact(pool_g, pool_o)
    hh.assert_attn_close(out_g, out_o, dtype)
