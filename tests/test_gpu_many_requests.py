"""Batches of many short requests: every suffix row finds its request, also next to requests without a suffix, and the rows cost
a launch little."""
import statistics

import pytest
import torch

import hip_harness as hh
from paper_2603_21257_amd import binding as cb
from paper_2603_21257_amd import workload as wl

pytestmark = pytest.mark.gpu


def slots(lens):
    return sum(-(-(p + s) // 16) for p, s in lens) + 9


@pytest.mark.parametrize("dtype,D,variant", [("bf16", 128, "3"), ("bf16", 128, "4"), ("bf16", 64, ""), ("f32", 64, "")])
@pytest.mark.parametrize("lens", [[(16 * (i % 5), (i * 7) % 40) for i in range(83)],
                                  [(0, 0), (16, 0), (0, 3)] + [(32, 1)] * 60 + [(48, 0), (0, 17), (16, 0)],
                                  [(16, 0)] * 64 + [(0, 5)], [(0, 64), (32, 40)] * 2 + [(0, 0)]])
def test_every_row_finds_its_request(dtype, D, variant, lens, monkeypatch):
    monkeypatch.setenv("CALVO_ATTN_VARIANT", variant)
    w = wl.make_custom(wl.Shape(1, 8, 2, D, dtype, slots(lens)), lens, seed=1000 + len(lens))
    print(f"[case] {dtype} D={D} variant={variant} requests={len(lens)}", flush=True)
    pool_g, out_g = hh.run_hip(w)
    pool_o, out_o = hh.run_oracle(w)
    hh.assert_pool_bit_exact(pool_g, pool_o)
    hh.assert_attn_close(out_g, out_o, dtype)


def layer_of(n, P, S, hq, hkv, with_suffix):
    """Median duration of one layer's launches for n requests, in ms."""
    s = wl.Shape(1, hq, hkv, 128, "bf16", slots([(P, S)] * n))
    w = wl.make_custom(s, [(P, S)] * n, seed=7, with_payload=False)
    mk = lambda *shape: wl.fill_normal_(torch.empty(shape, dtype=torch.bfloat16, device="cuda:0"), len(shape))
    pool, q, ks, vs = mk(s.pool_blocks, s.blk_elems), mk(n * S, hq, 128), mk(n * S, hkv, 128), mk(n * S, hkv, 128)
    out = torch.empty_like(q)
    torch.cuda.synchronize()
    ctx = cb.calvo_create(1, hq, hkv, 128, cb.CALVO_BF16, s.pool_blocks, pool)
    try:
        reqs = [cb.make_request(None, 0, r.table, r.n_prefix_blocks, S, r.n_prefix_blocks) for r in w.requests]
        batch = cb.calvo_batch_prepare(ctx, reqs, w.cu_suffix)
        times = []
        for _ in range(8):
            cb.calvo_prefill_attn_batch(ctx, batch, 0, q, ks if with_suffix else None, vs if with_suffix else None, out)
            times.append(cb.calvo_attn_kernel_ms(ctx, 0))
        cb.calvo_batch_destroy(batch)
    finally:
        cb.calvo_destroy(ctx)
    torch.cuda.empty_cache()
    return statistics.median(times[3:])


@pytest.mark.timing
@pytest.mark.parametrize("n,P,S,hq,hkv", [(256, 1024, 64, 32, 8), (250, 0, 16, 8, 8), (128, 1024, 256, 8, 8)])
def test_suffix_rows_cost_a_launch_little(n, P, S, hq, hkv):
    """A row finds its request in the logarithm of their number: 429 us with the rows and 375 without, 26 and 17.  Looked for one
    request after the other, they took 768 and 82.  Rows of more workgroups than the chip has room for go first: within the launch
    the last batch's took 325 us, 216 without."""
    without, with_rows = layer_of(n, P, S, hq, hkv, False), layer_of(n, P, S, hq, hkv, True)
    print(f"[case] {n} requests {P}+{S}: {with_rows * 1e3:.1f} us with the rows, {without * 1e3:.1f} without", flush=True)
    assert with_rows < 1.25 * without + 0.015
