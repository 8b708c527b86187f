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


# edges with register-resident sweeps, all of the largest class of line lengths
REGISTER = (3584, 3600, 3840, 3888, 3920, 4000, 4032)


def test_register_resident_edges_share_a_launch_with_none():
    # a group ordered by edge: its planes from the first on that may share a launch. A register-resident
    # edge between two others of its class, at either end, repeated, and alone
    count = _rule("_ZN2fr15mr_launch_countEPKii", ctypes.POINTER(ctypes.c_int), ctypes.c_int)
    default = _rule("_ZN2fr15mr_default_planEi", ctypes.c_int)
    default.restype = ctypes.c_uint
    run = lambda *edges: count((ctypes.c_int * len(edges))(*edges), len(edges))
    for e in REGISTER:
        assert default(e)
        assert run(2058, 2100, e, 4050) == 2
        assert run(e, 4050, 4050) == 1 and run(e, e, 4050) == 2 and run(e) == 1
        assert run(2058, e) == 1 and run(e, e, e) == 3
    assert run(2058, 3375, 3969, 4050) == 4
    # the classes of line lengths up to 2048 give the same bits in one launch, the largest does not
    assert run(250, 256, 257, 500, 1000, 2025) == 6 and run(250, 2058) == 1 and run(1000, 2025, 2058, 2100) == 2


def test_packed_plans_past_radix_16():
    past = _rule("_ZN2fr10mr_past_16Ej", ctypes.c_uint)
    past.restype = ctypes.c_bool
    pack = lambda *radices: sum(r << 5 * i for i, r in enumerate(radices))
    assert past(pack(18, 12, 18)) and past(pack(20, 10, 20)) and past(pack(2, 16, 28)) and past(pack(9, 17))
    assert not past(pack(16, 16, 14)) and not past(pack(9, 16, 14, 2)) and not past(pack(10, 10, 10)) and not past(0)
