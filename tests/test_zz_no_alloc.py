"""calvo_prefill_attn_noalloc (the entry point for callers that cannot allocate device memory)
against calvo_prefill_attn: same pool bytes, same attention output, on two calls in a row that
share the library's static device array - the second one smaller - and both against the oracle."""
import os

import numpy as np
import pytest

import hip_harness as hh
from paper_2603_21257_amd import binding as cb
from paper_2603_21257_amd import workload as wl

pytestmark = pytest.mark.gpu


def _both(w, **kw):
    pool_a, out_a = hh.run_hip(w, **kw)
    pool_n, out_n = hh.run_hip(w, attn_fn=cb.calvo_prefill_attn_noalloc, **kw)
    return (pool_a, out_a), (pool_n, out_n)


def _check(w, ref, new):
    hh.assert_pool_bit_exact(new[0], ref[0])
    # same kernels, same launch plan: the two entry points differ only in where descriptors and
    # partial results live, so the outputs agree to the bar of the parity tests (and in fact bit for bit)
    g = hh.orc.widen(new[1]) if new[1].dtype == np.uint16 else new[1].astype(np.float64)
    e = hh.orc.widen(ref[1]) if ref[1].dtype == np.uint16 else ref[1].astype(np.float64)
    tmx, tmean = hh.TOL[w.shape.dtype]
    d = np.abs(g - e)
    assert np.isfinite(g).all()
    assert d.max() <= tmx and d.mean() <= tmean, (d.max(), d.mean())
    pool_o, out_o = hh.run_oracle(w)
    hh.assert_pool_bit_exact(new[0], pool_o)
    hh.assert_attn_close(new[1], out_o, w.shape.dtype)


def test_noalloc_matches_prefill_attn_twice_second_smaller(monkeypatch):
    # first call: split tiles (partial results go through the static array), two requests
    monkeypatch.setenv("CALVO_ATTN_SPLITS", "3")
    shape = wl.Shape(2, 8, 2, 128, "bf16", 700)
    big = wl.make_custom(shape, [(4096, 70), (2048, 33)], seed=71)
    ref, new = _both(big)
    _check(big, ref, new)
    # second call, smaller, no cut tiles: stale descriptors and partial results of the first call
    # are still in the array and must not matter
    monkeypatch.delenv("CALVO_ATTN_SPLITS")
    small = wl.make_custom(wl.Shape(1, 8, 2, 128, "bf16", 64), [(256, 40)], seed=72)
    ref, new = _both(small)
    _check(small, ref, new)


def test_noalloc_fp32_path_and_repeat_in_one_context():
    # the packed-rows kernel (fp32 pool) has its descriptors and partial results in the same array
    w = wl.make_custom(wl.Shape(1, 8, 2, 64, "f32", 96), [(512, 50)], seed=73)
    ref, new = _both(w)
    _check(w, ref, new)


def test_noalloc_rejects_what_does_not_fit(monkeypatch):
    import torch
    monkeypatch.setenv("CALVO_ATTN_SPLITS", "8")
    shape = wl.Shape(1, 8, 2, 128, "bf16", 1200)
    w = wl.make_custom(shape, [(8192, 4096)], seed=74, with_payload=False)
    pool = torch.zeros((shape.pool_blocks * shape.blk_elems,), dtype=torch.bfloat16, device="cuda:0")
    q = torch.zeros((4096, 8, 128), dtype=torch.bfloat16, device="cuda:0")
    out = torch.full_like(q, 7.0)
    ctx = cb.calvo_create(1, 8, 2, 128, cb.CALVO_BF16, shape.pool_blocks, pool)
    try:
        r = w.requests[0]
        req = cb.make_request(None, 0, r.table, r.n_prefix_blocks, r.suffix_len, r.n_prefix_blocks)
        with pytest.raises(cb.CalvoError) as ei:
            cb.calvo_prefill_attn_noalloc(ctx, 0, q, None, None, out, [req], w.cu_suffix)
        assert ei.value.code == cb.CALVO_ENOMEM and "partial-result slots" in str(ei.value)
        torch.cuda.synchronize()
        assert bool((out == 7.0).all())          # nothing was queued
    finally:
        cb.calvo_destroy(ctx)


# (head layout, lengths): ragged batches whose best plan and whose plan with few, long pieces both need more partial
# results than the array holds on 256 CUs
RAGGED = [(32, 8, [(560, 3), (23936, 7), (5600, 33), (22976, 1486)]), (64, 8, [(7968, 434), (54432, 10), (9408, 41)]),
          (40, 8, [(9392, 2), (78240, 35)]), (48, 8, [(6608, 584), (5312, 8)]), (32, 8, [(0, 10), (43328, 105), (864, 115)]),
          (16, 2, [(9232, 711), (80, 706)]), (16, 8, [(0, 749), (4592, 1273), (448, 6)])]


@pytest.mark.parametrize("hq,hkv,lens", RAGGED)
def test_noalloc_takes_ragged_batches(hq, hkv, lens):
    import torch
    shape = wl.Shape(1, hq, hkv, 128, "bf16", sum(-(-(p + s) // 16) for p, s in lens) + 9)
    w = wl.make_custom(shape, lens, seed=75, with_payload=False)
    gen = torch.Generator(device="cuda:0").manual_seed(75)
    normal = lambda *n: torch.randn(n, generator=gen, dtype=torch.float32, device="cuda:0").to(torch.bfloat16)
    pool = normal(shape.pool_blocks, 2, 16, hkv, 128)
    q, ks, vs = normal(w.total_suffix, hq, 128), normal(w.total_suffix, hkv, 128), normal(w.total_suffix, hkv, 128)
    out = torch.full_like(q, float("nan"))
    torch.cuda.synchronize()
    ctx = cb.calvo_create(1, hq, hkv, 128, cb.CALVO_BF16, shape.pool_blocks, pool)
    try:
        reqs = [cb.make_request(None, 0, r.table, r.n_prefix_blocks, r.suffix_len, r.n_prefix_blocks) for r in w.requests]
        cb.calvo_prefill_attn_noalloc(ctx, 0, q, ks, vs, out, reqs, w.cu_suffix)
    finally:
        cb.calvo_destroy(ctx)
    view = hh.to_numpy_stored(pool, shape)                  # with the suffix rows
    got, qn = hh.to_numpy_stored(out, shape), hh.to_numpy_stored(q, shape)
    assert np.isfinite(hh.orc.widen(got)).all()
    for i, r in enumerate(w.requests):
        a, b = int(w.cu_suffix[i]), int(w.cu_suffix[i + 1])
        rows = sorted({0, (b - a) // 2, b - a - 1})
        want = hh.orc.prefill_attn_sampled(view, qn[a:b], r.table, r.prefix_len, r.suffix_len, 16, rows)
        hh.assert_attn_close(got[a:b][rows], want, "bf16")
