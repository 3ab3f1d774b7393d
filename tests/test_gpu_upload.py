"""Descriptor uploads around the size where a launch takes over from a copy (4096 words: about 1340 table entries with
their two-word offsets), through every entry point, and word counts that are not a multiple of four."""
import pytest

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
