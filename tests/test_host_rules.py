"""Host rules that choose how a call is launched, called in the built library (no GPU needed)."""

import ctypes

from paper_1806_06467_amd import fresnel as fb


def _rule(name, *argtypes):
    f = getattr(fb.lib(), name)
    f.argtypes, f.restype = argtypes, ctypes.c_int
    return f


def test_short_mft_products_fill_their_rounds():
    # a round is 256 blocks with a tile on each of their four SIMDs: of what the rounds of a square
    # output of every edge could do, at least half is done
    per_block = _rule("_ZN2fr16fold_short_tilesEii", ctypes.c_int, ctypes.c_int)
    up = lambda x, y: -(-x // y)
    for edge in range(1440, 8193):
        tiles, ftiles = up(edge // 2, 32), up(edge, 32)
        per = per_block(tiles, ftiles)
        assert 1 <= per <= tiles
        rounds = up(up(tiles, per) * ftiles, 256)
        assert 2 * tiles * ftiles >= rounds * 256 * up(per, 4) * 4, edge
