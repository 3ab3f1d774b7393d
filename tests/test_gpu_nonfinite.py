"""Infinities and NaNs in K, Q and V reach exactly the rows and columns that they reach in the oracle, and values near
the end of the element type's range do not overflow on the way."""
import numpy as np
import pytest

import hip_harness as hh
from paper_2603_21257_amd import workload as wl

pytestmark = pytest.mark.gpu


def stored(value, dtype):
    return np.uint16(np.float32(value).view(np.uint32) >> 16) if dtype == "bf16" else np.float32(value)


def assert_like_oracle(got_stored, want, dtype):
    got = hh.orc.widen(got_stored) if dtype == "bf16" else got_stored.astype(np.float64)
    for name, f in (("NaN", np.isnan), ("+inf", np.isposinf), ("-inf", np.isneginf)):
        bad = np.argwhere(f(got) != f(want))
        assert len(bad) == 0, f"{name} differs at {len(bad)} elements, first (layer, token, head, d) = {bad[0].tolist()}"
    ok = np.isfinite(want)
    d = np.abs(got[ok] - want[ok])
    tmx, tmean = hh.TOL[dtype]
    assert d.max() <= tmx and d.mean() <= tmean, (d.max(), d.mean())


def poisoned(shape, P, S, seed):
    """V: +inf at a cached token and -inf / NaN at two suffix tokens, in some columns only."""
    w = wl.make_custom(shape, [(P, S)], seed=seed)
    v = w.host_kv.reshape(shape.n_layers, w.host_blocks, 2, 16, shape.n_kv_heads, shape.head_dim)
    start = w.requests[0].host_block_start
    v[:, start + 2, 1, 7, :, ::4] = stored(np.inf, shape.dtype)
    w.v_suffix[:, 20, :, 2::4] = stored(-np.inf, shape.dtype)
    w.v_suffix[:, 30, :, ::8] = stored(-np.inf, shape.dtype)
    w.v_suffix[:, 30, :, 5] = stored(np.nan, shape.dtype)
    return w


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f32", 96), ("f32", 128), ("f32", 256), ("bf16", 40), ("bf16", 64),
                                     ("bf16", 96), ("bf16", 200), ("bf16", 256)])
@pytest.mark.parametrize("pieces", [1, 3])
@pytest.mark.parametrize("tile", ["1", "2"])
def test_v_of_packed_rows(dtype, D, pieces, tile, monkeypatch):
    monkeypatch.setenv("CALVO_ROWS_TILE", tile)
    if pieces > 1:
        monkeypatch.setenv("CALVO_ATTN_SPLITS", str(pieces))
    s = wl.Shape(1, 6, 2, D, dtype, 40)
    w = poisoned(s, 400, 45, seed=800 + D)
    print(f"[case] {dtype} D={D} pieces={pieces} tile={tile}", flush=True)
    _, got = hh.run_hip(w)
    with np.errstate(invalid="ignore"):
        _, want = hh.run_oracle(w)
    assert_like_oracle(got, want, dtype)


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f32", 128), ("f32", 256), ("bf16", 64), ("bf16", 96), ("bf16", 256)])
@pytest.mark.parametrize("value,columns", [(1e35, slice(None)), (1e32, slice(0, 1))])
@pytest.mark.parametrize("pieces", [1, 2])
@pytest.mark.parametrize("tile", ["1", "2"])
def test_large_v_under_rising_scores(dtype, D, value, columns, pieces, tile, monkeypatch):
    """All scores are 0 up to a token from which on they are 15 powers of two higher.  The softmax reference lags by up
    to 16 powers of two; sums of V taken with weights of 2^15 would leave the range where the result does not - in one
    wave, or (1e32 in one column) where the waves' sums are added."""
    monkeypatch.setenv("CALVO_ROWS_TILE", tile)
    monkeypatch.setenv("CALVO_ATTN_SPLITS", str(pieces))
    P, S = 1024, 20
    s = wl.Shape(1, 4, 2, D, dtype, (P + S) // 16 + 9)
    w = wl.make_custom(s, [(P, S)], seed=903)
    w.q[...] = stored(1.0, dtype)
    first = w.requests[0].host_block_start
    kv = w.host_kv.reshape(1, w.host_blocks, 2, 16, 2, D)[0, first:first + P // 16]
    kv[:, 0] = stored(0.0, dtype)
    kv[16:, 0, :, :, 0] = stored(np.round(15 * np.log(2) * np.sqrt(D)), dtype)
    w.k_suffix[...] = stored(0.0, dtype)
    factor = np.ones(D)
    factor[columns] = value
    for v in (kv[:, 1], w.v_suffix):
        x = (np.abs(hh.orc.widen(v)) * factor).astype(np.float32)
        v[...] = (x.view(np.uint32) >> 16).astype(np.uint16) if dtype == "bf16" else x
    _, got = hh.run_hip(w)
    _, want = hh.run_oracle(w)
    g = hh.orc.widen(got) if dtype == "bf16" else got.astype(np.float64)
    tmx, tmean = hh.TOL[dtype]
    d = np.abs(g / factor - want / factor)
    assert np.isfinite(g).all() and d.max() <= tmx and d.mean() <= tmean, (d.max(), d.mean())


@pytest.mark.parametrize("pieces", [1, 3])
def test_next_score_in_32_bits_far_below_zero(pieces, monkeypatch):
    """The scores of later keys are the next value in 32 bits above the earlier ones and 131 powers of two higher.  The score at
    which the softmax reference moves is a product that rounds: rounded up to theirs, the weights against the earlier
    reference would be finite and their sum not (V is so small that the sums of it are)."""
    monkeypatch.setenv("CALVO_ATTN_SPLITS", str(pieces))
    P, S, D = 1024, 20, 128
    w = wl.make_custom(wl.Shape(1, 4, 2, D, "f32", (P + S) // 16 + 9), [(P, S)], seed=905)
    w.q[...] = 0.0
    w.q[..., 0] = 1.0
    first = w.requests[0].host_block_start
    kv = w.host_kv.reshape(1, w.host_blocks, 2, 16, 2, D)[0, first:first + P // 16]
    kv[:16, 0, :, :, 0] = -16660231168.0
    kv[16:, 0, :, :, 0] = w.k_suffix[..., 0] = -16660230144.0
    kv[:, 1] *= np.float32(2.0 ** -30)
    w.v_suffix *= np.float32(2.0 ** -30)
    _, got = hh.run_hip(w)
    _, want = hh.run_oracle(w)
    d = np.abs(got.astype(np.float64) - want) * 2.0 ** 30
    tmx, tmean = hh.TOL["f32"]
    assert np.isfinite(got).all() and d.max() <= tmx and d.mean() <= tmean, (d.max(), d.mean())


@pytest.mark.parametrize("variant", ["3", "4"])
@pytest.mark.parametrize("value,columns", [(1e35, slice(None)), (1e33, slice(0, 1))])
@pytest.mark.parametrize("P,S,rise", [
    (0, 64, (32, 33)), (0, 300, (33, 300)), (48, 200, (64, 70)),                         # diagonal
    (96, 5, (64, 96)), (352, 5, (320, 352)),                                             # drain
    (128, 5, (32, 33)), (160, 64, (64, 96)), (1024, 20, (256, 1024)), (4096, 70, (3000, 3001))])
@pytest.mark.parametrize("pieces", [0, 2])
def test_large_v_under_rising_scores_of_128_wide_heads(variant, value, columns, P, S, rise, pieces, monkeypatch):
    """Scores of the keys `rise` are 12 powers of two above the others (eight of them stay below the 2^16 at which the
    reference moves), wherever they lie: in the pipelined steps, behind them or on the diagonal."""
    monkeypatch.setenv("CALVO_ATTN_VARIANT", variant)
    if pieces:
        monkeypatch.setenv("CALVO_ATTN_SPLITS", str(pieces))
    D = 128
    w = wl.make_custom(wl.Shape(1, 4, 1, D, "bf16", (P + S) // 16 + 9), [(P, S)], seed=904)
    w.q[...] = stored(1.0, "bf16")
    first = w.requests[0].host_block_start
    kv = w.host_kv.reshape(1, w.host_blocks, 2, 16, 1, D)[0, first:first + P // 16]
    kv[:, 0] = 0
    w.k_suffix[...] = 0
    high = stored(np.round(12 * np.log(2) * np.sqrt(D)), "bf16")
    for t in range(*rise):
        if t < P:
            kv[t // 16, 0, t % 16, :, 0] = high
        else:
            w.k_suffix[0, t - P, :, 0] = high
    factor = np.ones(D)
    factor[columns] = value
    for v in (kv[:, 1], w.v_suffix):
        x = (np.abs(hh.orc.widen(v)) * factor).astype(np.float32)
        v[...] = (x.view(np.uint32) >> 16).astype(np.uint16)
    _, got = hh.run_hip(w)
    _, want = hh.run_oracle(w)
    g = hh.orc.widen(got)
    tmx, tmean = hh.TOL["bf16"]
    d = np.abs(g / factor - want / factor)
    assert np.isfinite(g).all() and d.max() <= tmx and d.mean() <= tmean, (d.max(), d.mean())


def long_one_token(seed, P=8192):
    s = wl.Shape(1, 8, 2, 128, "bf16", P // 16 + 9)
    w = wl.make_custom(s, [(P, 1)], seed=seed)
    first = w.requests[0].host_block_start
    return w, w.host_kv.reshape(1, w.host_blocks, 2, 16, 2, 128)[0, first:first + P // 16]


@pytest.mark.parametrize("tokens", [slice(5, 6), slice(0, 1024), slice(7000, 7001)])
@pytest.mark.parametrize("pieces", [0, 1])
def test_nan_score_in_a_piece_of_a_cut_context(tokens, pieces, monkeypatch):
    """One token over 8K cached ones: the planner cuts the context, the pieces are merged.  A NaN in K is in no piece's
    sum alone: the whole row is NaN, as in a launch that is not cut."""
    if pieces:
        monkeypatch.setenv("CALVO_ATTN_SPLITS", str(pieces))
    w, kv = long_one_token(901)
    idx = np.arange(8192)[tokens]
    kv[idx // 16, 0, idx % 16, 1, 3] = stored(np.nan, "bf16")        # KV head 1: query heads 4..7
    _, got = hh.run_hip(w)
    with np.errstate(invalid="ignore"):
        _, want = hh.run_oracle(w)
    assert np.isnan(want[0, 0, 4:]).all()
    assert_like_oracle(got, want, "bf16")


def test_infinite_v_behind_a_weight_that_underflows_in_the_merge():
    """V of an early token is infinite in some columns and a late token's score is 300 powers of two above the others:
    the early piece's weight in the merge is 0 in 32 bits, its infinities are not: those columns are not finite."""
    w, kv = long_one_token(902)
    kv[0, 1, 5, 0, ::4] = stored(np.inf, "bf16")
    q = hh.orc.widen(w.q)[0, 0, 0].astype(np.float32)                # query head 0
    k = (q * np.float32(300 * np.log(2) * np.sqrt(128.0) / np.dot(q, q))).astype(np.float32)
    kv[8000 // 16, 0, 0, 0] = (k.view(np.uint32) >> 16).astype(np.uint16)
    _, got = hh.run_hip(w)
    _, want = hh.run_oracle(w)
    g = hh.orc.widen(got)[0, 0, 0]
    assert not np.isfinite(g[::4]).any()
    cols = np.arange(128) % 4 != 0
    assert np.abs(g[cols] - want[0, 0, 0][cols]).max() <= hh.TOL["bf16"][0]
