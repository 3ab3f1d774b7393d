"""calvo_attn_kernel_ms: the kernels' own clock, for every kernel and for launches that are merged or follow chunks."""
import time

import pytest
import torch

from paper_2603_21257_amd import binding as cb
from paper_2603_21257_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _give_memory_back():
    yield
    torch.cuda.empty_cache()          # other files count on large tensors being allocations of their own


@pytest.mark.parametrize("hq,D,dtype,P,S", [(8, 64, "f32", 1024, 40), (8, 64, "bf16", 4096, 3), (8, 128, "bf16", 16384, 8),
                                            (8, 128, "bf16", 4096, 1024), (10, 128, "bf16", 32768, 200)])
def test_duration_of_the_latest_launch(hq, D, dtype, P, S):
    s = wl.Shape(2, hq, 2, D, dtype, (P + S) // 16 + 8)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    mk = lambda *shape: torch.randn(shape, device="cuda:0").to(dt)
    pool, q, ks, vs = mk(2, s.pool_blocks, s.blk_elems), mk(S, hq, D), mk(S, 2, D), mk(S, 2, D)
    out = torch.empty_like(q)
    r = wl.single_request(s, P, S, 5)[0]
    torch.cuda.synchronize()
    ctx = cb.calvo_create(2, hq, 2, D, cb.CALVO_BF16 if dtype == "bf16" else cb.CALVO_F32, s.pool_blocks, pool)
    try:
        req = cb.make_request(None, 0, r.table, r.n_prefix_blocks, S, r.n_prefix_blocks)
        with pytest.raises(cb.CalvoError) as ei:
            cb.calvo_attn_kernel_ms(ctx, 1)
        assert ei.value.code == cb.CALVO_ENOTREADY
        for _ in range(5):
            t = time.perf_counter()
            cb.calvo_prefill_attn(ctx, 1, q, ks, vs, out, [req], [0, S])
            ms = cb.calvo_attn_kernel_ms(ctx, 1)
            wall = (time.perf_counter() - t) * 1e3
            assert 0 < ms < wall                     # inside the call's own wall time, also on repetition
            assert ms < 50
        with pytest.raises(cb.CalvoError):
            cb.calvo_attn_kernel_ms(ctx, 0)          # nothing was queued for that layer
    finally:
        cb.calvo_destroy(ctx)


@pytest.mark.timing
@pytest.mark.parametrize("hq,hkv,D,dtype,P,S,pieces", [(32, 8, 128, "bf16", 61440, 4096, 0), (32, 8, 128, "bf16", 4096, 1024, 64),
                                                       (8, 2, 256, "f32", 8192, 2048, 0), (8, 2, 64, "bf16", 512, 2048, 16)])
def test_agrees_with_events(hq, hkv, D, dtype, P, S, pieces, monkeypatch):
    """Against a pair of events on the compute stream, which have the launches' own start and end on top (30 us at most):
    launches of several milliseconds, and launches of which the merge of many pieces is the larger part."""
    if pieces:
        monkeypatch.setenv("CALVO_ATTN_SPLITS", str(pieces))
    s = wl.Shape(1, hq, hkv, D, dtype, (P + S) // 16 + 8)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    mk = lambda *shape: torch.randn(shape, device="cuda:0").to(dt)
    pool, q = mk(1, s.pool_blocks, s.blk_elems), mk(S, hq, D)
    out = torch.empty_like(q)
    r = wl.single_request(s, P, S, 5)[0]
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    ctx = cb.calvo_create(1, hq, hkv, D, cb.CALVO_BF16 if dtype == "bf16" else cb.CALVO_F32, s.pool_blocks, pool,
                          compute_stream=stream.cuda_stream)
    try:
        req = cb.make_request(None, 0, r.table, r.n_prefix_blocks, S, r.n_prefix_blocks)
        got = []
        for _ in range(5):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record(stream)
            cb.calvo_prefill_attn(ctx, 0, q, None, None, out, [req], [0, S])
            e1.record(stream)
            ms = cb.calvo_attn_kernel_ms(ctx, 0)
            e1.synchronize()
            got.append((ms, e0.elapsed_time(e1)))
        print(got, flush=True)
        ms, ev = sorted(got, key=lambda x: x[1] - x[0])[0]
        assert 0.98 * ev - 0.03 <= ms <= ev, got
    finally:
        cb.calvo_destroy(ctx)


@pytest.mark.timing
def test_waits_for_the_layer_that_is_asked_for():
    """Layer 0's launch, then 60 ms of other layers' on the compute stream and of the default stream's work: the time of
    layer 0 is there before either is done."""
    P, S = 49152, 4096
    s = wl.Shape(2, 32, 8, 128, "bf16", (P + S) // 16 + 8)
    mk = lambda *shape: torch.randn(shape, device="cuda:0", dtype=torch.bfloat16)
    pool, q, ks, vs = mk(2, s.pool_blocks, s.blk_elems), mk(S, 32, 128), mk(S, 8, 128), mk(S, 8, 128)
    out, a, b = torch.empty_like(q), mk(8192, 8192), mk(8192, 8192)
    r = wl.single_request(s, P, S, 5)[0]
    torch.mm(a, b)                                       # its library is loaded before, not while the launches run
    torch.cuda.synchronize()
    ctx = cb.calvo_create(2, 32, 8, 128, cb.CALVO_BF16, s.pool_blocks, pool)
    try:
        req = cb.make_request(None, 0, r.table, r.n_prefix_blocks, S, r.n_prefix_blocks)
        run = lambda l: cb.calvo_prefill_attn(ctx, l, q, ks, vs, out, [req], [0, S])
        run(0)
        first = cb.calvo_attn_kernel_ms(ctx, 0)
        run(0)
        for _ in range(20):
            run(1)
            torch.mm(a, b)
        ms = cb.calvo_attn_kernel_ms(ctx, 0)
        t = time.perf_counter()
        torch.cuda.synchronize()
        rest = (time.perf_counter() - t) * 1e3
        print(rest, first, ms, flush=True)
        assert rest > 10 * first                         # most of the twenty are still to come
    finally:
        cb.calvo_destroy(ctx)
