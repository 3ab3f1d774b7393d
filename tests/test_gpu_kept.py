"""The batch that calvo_prefill_attn keeps between calls is found by content: the same array objects with other contents
are another batch, a bad table is refused after a good one, and calls of different kinds may alternate."""
import numpy as np
import pytest
import torch

import hip_harness as hh
from paper_2603_21257_amd import binding as cb
from paper_2603_21257_amd import workload as wl

pytestmark = pytest.mark.gpu


class Case:
    def __init__(self, dtype, D, lens, seed):
        s = self.s = wl.Shape(1, 8, 2, D, dtype, sum(-(-(p + q) // 16) for p, q in lens) + 40)
        self.w = wl.make_custom(s, lens, seed=seed)
        dev, dt = torch.device("cuda:0"), hh.torch_dtype(s)
        self.pool = hh.to_torch(hh.sentinel_pool_np(s), s, dev)
        self.host = hh.to_torch(self.w.host_kv, s, pin=True)
        self.q, self.ks, self.vs = (hh.to_torch(a, s, dev) for a in (self.w.q, self.w.k_suffix, self.w.v_suffix))
        self.out = torch.empty((1, self.w.total_suffix, 8, D), dtype=dt, device=dev)
        torch.cuda.synchronize()
        self.ctx = cb.calvo_create(1, 8, 2, D, cb.CALVO_BF16 if dtype == "bf16" else cb.CALVO_F32, s.pool_blocks, self.pool)
        self.reqs = hh.make_requests(self.w, self.host)
        cb.calvo_kv_ingest(self.ctx, self.reqs, 0, 1)

    def run(self, fn=cb.calvo_prefill_attn):
        self.out.fill_(float("nan"))
        torch.cuda.synchronize()
        fn(self.ctx, 0, self.q[0], self.ks[0], self.vs[0], self.out[0], self.reqs, self.w.cu_suffix)
        torch.cuda.synchronize()
        return hh.to_numpy_stored(self.out, self.s)


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("f32", 64)])
def test_tables_changed_in_place_are_another_batch(dtype, D):
    c = Case(dtype, D, [(96, 20), (64, 5)], seed=51)
    try:
        _, want = hh.run_oracle(c.w)
        for fn in (cb.calvo_prefill_attn, cb.calvo_prefill_attn, cb.calvo_prefill_attn_noalloc, cb.calvo_prefill_attn):
            hh.assert_attn_close(c.run(fn), want, dtype)
        # the first request's prefix moves to free slots: same array object, other contents
        table = c.reqs[0]._keep
        free = np.setdiff1d(np.arange(c.s.pool_blocks), np.concatenate([r._keep for r in c.reqs]))[:3].astype(np.int32)
        old = table[:3].copy()
        c.pool[0][torch.from_numpy(free.astype(np.int64)).cuda()] = c.pool[0][torch.from_numpy(old.astype(np.int64)).cuda()]
        c.pool[0][torch.from_numpy(old.astype(np.int64)).cuda()] = 0
        table[:3] = free
        hh.assert_attn_close(c.run(), want, dtype)
        hh.assert_attn_close(c.run(cb.calvo_prefill_attn_noalloc), want, dtype)
        # a slot outside the pool, one that appears twice: refused although the rest was checked before
        for bad in (c.s.pool_blocks, int(table[1])):
            table[0] = bad
            with pytest.raises(cb.CalvoError) as ei:
                c.run()
            assert ei.value.code == cb.CALVO_EINVAL
        table[0] = free[0]
        hh.assert_attn_close(c.run(), want, dtype)
        # a wrong cu_suffix is refused too
        good = c.w.cu_suffix
        c.w.cu_suffix = good + np.array([0, 1, 1], np.int32)
        with pytest.raises(cb.CalvoError):
            c.run()
        c.w.cu_suffix = good
        hh.assert_attn_close(c.run(), want, dtype)
    finally:
        cb.calvo_destroy(c.ctx)


def test_forced_shapes_are_seen_by_a_kept_batch(monkeypatch):
    c = Case("bf16", 128, [(320, 70)], seed=52)
    try:
        _, want = hh.run_oracle(c.w)
        for variant in ("3", "4", "3", ""):
            monkeypatch.setenv("CALVO_ATTN_VARIANT", variant)
            hh.assert_attn_close(c.run(), want, "bf16")
            kernel, _ = cb.calvo_attn_kernel_info(c.ctx, 0)
            assert not variant or kernel == int(variant)
    finally:
        cb.calvo_destroy(c.ctx)


PREFILL, NOALLOC = cb.calvo_prefill_attn, cb.calvo_prefill_attn_noalloc


@pytest.mark.parametrize("lens", [(1024, 4096), (7648, 3284)])
@pytest.mark.parametrize("calls", [(NOALLOC,), (PREFILL, NOALLOC), (NOALLOC, PREFILL, NOALLOC)])
def test_plans_beyond_the_fixed_array(lens, calls):
    """The best plans of these batches have more partial results than the fixed-size array holds; the allocation-free
    entry point runs them with longer pieces, whatever call was made before."""
    c = Case("bf16", 128, [lens], seed=53)
    try:
        for fn in calls:
            out = c.run(fn)[0]
            pool = hh.to_numpy_stored(c.pool, c.s)
            rows = [0, 31, 32, 1500, lens[1] - 1]
            want = hh.orc.prefill_attn_sampled(pool[0].reshape(-1, 2, 16, 2, 128), c.w.q[0], c.w.requests[0].table, *lens, 16, rows)
            assert np.isfinite(hh.orc.widen(out)).all()
            hh.assert_attn_close(out[rows], want, "bf16")
    finally:
        cb.calvo_destroy(c.ctx)
