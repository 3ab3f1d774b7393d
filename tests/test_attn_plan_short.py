"""Cuts of short contexts and of batches whose tiles differ in length (host code, no GPU)."""
import numpy as np
import pytest

from paper_2603_21257_amd import binding as cb

CUS = 256


def pieces_by_tile(hq, hkv, lens):
    items = cb.calvo_attn_plan_items(hq, hkv, CUS, [p // 16 for p, _ in lens], [s for _, s in lens])
    tiles = {}
    for req, tile, b, e, n, _ in items:
        tiles.setdefault((req, tile), []).append((int(b), int(e), int(n)))
    return tiles


@pytest.mark.parametrize("P", [512, 1024, 2048, 4096, 8192, 16384, 28096, 65536])
@pytest.mark.parametrize("S", [1, 28, 64])
def test_pieces_are_not_shorter_than_the_floor(P, S):
    for pieces in pieces_by_tile(32, 8, [(P, S)]).values():
        n_sub = pieces[-1][1]
        floor = min(48, max(8, n_sub // 32))
        for b, e, n in pieces[:-1]:                # the last piece is what is left
            assert e - b >= min(floor, n_sub)
    if 2048 <= P <= 16384:
        assert len(pieces) >= 6                    # an 8B-shape tile is eight workgroups on 256 CUs otherwise


def test_a_long_context_does_not_cut_the_short_ones_beside_it():
    tiles = pieces_by_tile(40, 8, [(3568, 164), (1648, 171), (1264, 381), (38480, 4)])
    assert len(tiles[(3, 0)]) > 4
    assert all(len(p) == 1 for (req, _), p in tiles.items() if req in (1, 2))


@pytest.mark.parametrize("seed", range(6))
def test_piece_lengths_are_alike_over_a_mixed_batch(seed):
    """No piece of a cut tile is longer than twice the longest tile's pieces, no tile has more pieces than that one."""
    rng = np.random.default_rng(5100 + seed)
    lens = [(int(rng.integers(0, 4000)) * 16, int(rng.integers(1, 300))) for _ in range(int(rng.integers(2, 6)))]
    tiles = pieces_by_tile(32, 8, lens)
    longest = max(tiles.values(), key=lambda p: p[-1][1])
    assert all(len(p) <= len(longest) for p in tiles.values())
    step = max(e - b for b, e, _ in longest)
    assert all(e - b <= 2 * step + 8 for p in tiles.values() for b, e, _ in p)


@pytest.mark.parametrize("hq,hkv,lens", [(16, 8, [(1648, 7)]), (64, 8, [(1488, 27)]), (64, 8, [(128, 1), (1680, 10)]),
                                         (32, 8, [(1616, 2), (160, 3), (0, 212), (240, 53)])])
def test_contexts_between_1k_and_2k_are_cut(hq, hkv, lens):
    """8 to 32 workgroups that walk some 50 sub-tiles each take twice the time of six times as many."""
    tiles = pieces_by_tile(hq, hkv, lens)
    assert max(len(p) for p in tiles.values()) >= 4
