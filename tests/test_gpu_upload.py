"""Descriptor uploads around the size where a launch takes over from a copy (4096 words: about 1340 table entries with
their two-word offsets), through every entry point, and word counts that are not a multiple of four."""
import numpy as np
import pytest
import torch

import hip_harness as hh
from paper_2603_21257_amd import binding as cb
from paper_2603_21257_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prefix_blocks", [1318, 1319, 1325, 1326, 1501])
@pytest.mark.parametrize("kw", [dict(), dict(prepared=True), dict(attn_fn=cb.calvo_prefill_attn_noalloc)])
def test_large_tables(prefix_blocks, kw):
    w = wl.make_custom(wl.Shape(1, 4, 1, 128, "bf16", prefix_blocks + 20), [(16 * prefix_blocks, 3)], seed=prefix_blocks)
    print(f"[case] prefix_blocks={prefix_blocks} kw={kw}", flush=True)
    pool_g, out_g = hh.run_hip(w, **kw)
    pool_o, out_o = hh.run_oracle(w)
    hh.assert_pool_bit_exact(pool_g, pool_o)
    hh.assert_attn_close(out_g, out_o, "bf16")


@pytest.mark.parametrize("how", ["call", "noalloc", "batch"])
def test_uploads_in_turn_read_what_the_host_wrote_last(how):
    """Six batches of the same lengths with tables of their own, forty calls in turn without a wait in between: the
    page-locked buffers that the uploads read are written again and again while the stream runs."""
    P, S, n = 16 * 1400, 3, 6
    s = wl.Shape(1, 4, 1, 128, "bf16", 3000)
    pool = torch.randn((1, s.pool_blocks, s.blk_elems), device="cuda:0").bfloat16()
    q = torch.randn((S, 4, 128), device="cuda:0").bfloat16()
    out = torch.zeros((40, S, 4, 128), dtype=torch.bfloat16, device="cuda:0")
    want = torch.zeros((n, S, 4, 128), dtype=torch.bfloat16, device="cuda:0")
    rng = np.random.default_rng(77)
    tables = [rng.permutation(s.pool_blocks)[:1401].astype(np.int32) for _ in range(n)]
    reqs = [[cb.make_request(None, 0, t, 1400, S, 1400)] for t in tables]
    torch.cuda.synchronize()
    ctx = cb.calvo_create(1, 4, 1, 128, cb.CALVO_BF16, s.pool_blocks, pool)
    try:
        for i in range(n):
            cb.calvo_prefill_attn(ctx, 0, q, None, None, want[i], reqs[i], [0, S])
            cb.calvo_attn_kernel_ms(ctx, 0)                  # waits for the launch
        for i in range(40):
            if how == "batch":
                b = cb.calvo_batch_prepare(ctx, reqs[i % n], [0, S])
                cb.calvo_prefill_attn_batch(ctx, b, 0, q, None, None, out[i])
                cb.calvo_batch_destroy(b)                    # its buffers go to the next batch
            else:
                fn = cb.calvo_prefill_attn if how == "call" else cb.calvo_prefill_attn_noalloc
                fn(ctx, 0, q, None, None, out[i], reqs[i % n], [0, S])
    finally:
        cb.calvo_destroy(ctx)
    torch.cuda.synchronize()
    assert len({w.float().sum().item() for w in want}) == n
    bad = [i for i in range(40) if not torch.equal(out[i], want[i % n])]
    assert not bad, bad
