"""GPU parity of mft_forward / mft_adjoint against the FP64 oracle (ragged shapes, windows,
masks, Babinet alpha/beta) and the Airy closed form."""

import numpy as np
import pytest
import torch
from scipy.special import j1

import oracle
from paper_1806_06467_amd import fresnel as fb
from paper_1806_06467_amd import synth
from tests.gpu_common import banner, f32, forced_gemm_tile, rel_l2, to_gpu, to_np

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.mark.parametrize("n_in,m,n_d,du", [(512, 128, 256.0, 0.25), (100, 37, 40.0, 0.61),
                                            (1024, 256, 256.0, 8 / 256), (64, 512, 32.0, 0.25),
                                            (1000, 130, 500.0, 0.3)])
def test_mft_forward_matches_oracle(n_in, m, n_d, du):
    banner(f"mft_forward {n_in}->{m}")
    e = synth.random_field(n_in, n_in + m)
    got = to_np(fb.mft_forward(to_gpu(e), n_d, m, du))
    ref = oracle.mft(f32(e), n_d, m, du)
    assert rel_l2(got, ref) <= TOL
    assert rel_l2(np.abs(got) ** 2, np.abs(ref) ** 2) <= TOL


def test_mft_forward_window_and_mask():
    n, nd, m, du = 512, 200, 96, 0.4
    big = synth.random_field(n, 9)
    off = (n - nd) // 2
    mask = synth.occulter_spot(m, du, 3.0)
    t = to_gpu(big)
    win = t[off:off + nd, off:off + nd]
    got = to_np(fb.mft_forward(win, float(nd), m, du, mask=to_gpu(mask, torch.float32)))
    ref = mask * oracle.mft(f32(big)[off:off + nd, off:off + nd], float(nd), m, du)
    assert rel_l2(got, ref) <= TOL


@pytest.mark.parametrize("m,n_out,n_d,du", [(128, 512, 256.0, 0.25), (37, 100, 40.0, 0.61),
                                             (256, 1024, 1024.0, 8 / 256)])
def test_mft_adjoint_matches_oracle(m, n_out, n_d, du):
    banner(f"mft_adjoint {m}->{n_out}")
    eb = synth.random_field(m, m + n_out)
    got = to_np(fb.mft_adjoint(to_gpu(eb), n_d, n_out, du))
    ref = oracle.mft_adjoint(f32(eb), n_d, n_out, du)
    assert rel_l2(got, ref) <= TOL


def test_mft_adjoint_babinet_into_window():
    # out_window = lyot * (out_window - MFT^H(eb)): alpha = -1, beta = 1, mask = lyot
    n, nd, m, du = 640, 256, 128, 8 / 128
    plane = synth.random_field(n, 11)
    eb = synth.random_field(m, 12)
    lyot = synth.lyot_stop(nd, 0.9)
    off = (n - nd) // 2
    t = to_gpu(plane)
    win = t[off:off + nd, off:off + nd]
    fb.mft_adjoint(to_gpu(eb), float(nd), nd, du, alpha=-1.0, beta=1.0,
                   mask=to_gpu(lyot, torch.float32), out=win)
    got = to_np(t)
    ref = f32(plane).copy()
    ref[off:off + nd, off:off + nd] = lyot * (ref[off:off + nd, off:off + nd]
                                              - oracle.mft_adjoint(f32(eb), float(nd), nd, du))
    assert rel_l2(got, ref) <= TOL


def test_occulter_mft_full_size():
    n, nd, m, du = 4096, 1024.0, 256, 8 / 256
    banner("occulter mft 4096 -> 256")
    e = synth.random_field(n, 4)
    got = to_np(fb.mft_forward(to_gpu(e), nd, m, du))
    ref = oracle.mft(f32(e), nd, m, du)
    assert rel_l2(got, ref) <= TOL


def test_airy_256_aperture_on_gpu():
    ap = synth.circular_aperture(512, 128.0)
    got = to_np(fb.mft_forward(to_gpu(ap), 256.0, 128, 0.25))
    assert abs(got[64, 64] - 0.25 / 256 * 51429) <= 1e-5 * 50.2236
    rho = np.abs((np.arange(128) - 64) * 0.25)
    with np.errstate(invalid="ignore", divide="ignore"):
        airy = np.where(rho > 0, 2 * j1(np.pi * rho) / (np.pi * rho), 1.0)
    core = rho <= 3.0
    cut = np.abs(got[64, :]) / abs(got[64, 64])
    assert np.max(np.abs(cut - np.abs(airy))[core]) <= 1.5e-3


@pytest.mark.parametrize("tile,split", [(0, 0), (1, 0), (2, 0), (3, 0), (4, 0), (5, 0), (6, 0), (0, 1),
                                        (1, 3), (2, 16), (3, 7), (4, 5), (5, 2), (6, 3)])
def test_every_gemm_tile_configuration_matches_oracle(tile, split, tmp_path):
    # force one tile configuration (4 and 5: three real products per complex step; 6: the same on
    # bfloat16 pieces of the operands) and split-K
    # factor (0: the tile's default) on all four GEMMs
    # of a ragged forward and adjoint MFT (through the autotuner's file format) and check both
    # transforms against the oracle; 16 slices of K = 130 leave trailing slices empty
    n, m, n_d, du = 1000, 130, 500.0, 0.3
    banner(f"mft with GEMM tile configuration {tile}, split {split}")
    shapes = [(n, m, n, 0, 1), (m, m, n, 0, 0), (m, n, m, 0, 1), (n, n, m, 0, 0)]
    f = tmp_path / "tiles.txt"
    f.write_text("".join("gemm %d %d %d %d %d %d %d\n" % (s + (tile, split)) for s in shapes))
    fb.autotune_load(str(f))
    e = synth.random_field(n, 31)
    got = to_np(fb.mft_forward(to_gpu(e), n_d, m, du))
    assert rel_l2(got, oracle.mft(f32(e), n_d, m, du)) <= TOL
    eb = synth.random_field(m, 32)
    got = to_np(fb.mft_adjoint(to_gpu(eb), n_d, n, du))
    assert rel_l2(got, oracle.mft_adjoint(f32(eb), n_d, n, du)) <= TOL


def test_autotune_file_refuses_a_split_beyond_the_limit(tmp_path):
    f = tmp_path / "bad.txt"
    f.write_text("gemm 1000 130 1000 0 1 0 17\n")
    with pytest.raises(fb.FrError):
        fb.autotune_load(str(f))
    f.write_text("gemm_default 7 0\n")   # no tile configuration 7
    with pytest.raises(fb.FrError):
        fb.autotune_load(str(f))


def test_default_gemm_choice_applies_to_untuned_shapes(tmp_path):
    # a default tile / split for every shape without its own line: the three-product tile on a
    # ragged pair of transforms, then back to the choice by shape
    n, m, n_d, du = 700, 90, 350.0, 0.45
    f = tmp_path / "default.txt"
    f.write_text("gemm_default 4 3\n")
    fb.autotune_load(str(f))
    try:
        e = synth.random_field(n, 41)
        got = to_np(fb.mft_forward(to_gpu(e), n_d, m, du))
        assert rel_l2(got, oracle.mft(f32(e), n_d, m, du)) <= TOL
        eb = synth.random_field(m, 42)
        got = to_np(fb.mft_adjoint(to_gpu(eb), n_d, n, du))
        assert rel_l2(got, oracle.mft_adjoint(f32(eb), n_d, n, du)) <= TOL
        saved = tmp_path / "saved.txt"
        fb.autotune_save(str(saved))
        assert "gemm_default 4 3" in saved.read_text()
    finally:
        f.write_text("gemm_default -1 0\n")
        fb.autotune_load(str(f))


def test_bfloat16_split_tile_on_8192_field(tmp_path):
    # the bfloat16-split tile reads the 512 MiB field through 32-bit buffer offsets: the
    # occulter MFT of an 8192^2 field (the large train's grid) against the oracle, every GEMM on
    # that tile
    n, nd, m, du = 8192, 2048.0, 256, 8 / 256
    banner("bfloat16-split tile: occulter mft 8192 -> 256")
    with forced_gemm_tile(6, tmp_path):
        e = synth.random_field(n, 21)
        got = to_np(fb.mft_forward(to_gpu(e), nd, m, du))
    ref = oracle.mft(f32(e), nd, m, du)
    assert rel_l2(got, ref) <= TOL


# edges of the folded products: lengths 1 to 3 (no pair, an unpaired first element), 63 / 64 / 65
# outputs and 127 to 130 inputs (32-wide tiles, 64-pair stages, odd and even), several stages
@pytest.mark.parametrize("n,m", [(1, 1), (2, 3), (3, 2), (64, 65), (65, 64), (127, 63), (128, 129), (129, 128),
                                 (130, 257), (258, 130), (385, 66), (1030, 34)])
def test_folded_products_at_tile_edges(n, m):
    # float32 roundings in a row: the fold and the product T of each axis, the result, the matrix
    # pieces (2^-25 and 2^-23 left out) and eight float32 sums per 128 pairs: below 24 x 2^-24
    banner(f"folded mft {n} <-> {m}")
    n_d, du = max(1.0, 0.4 * n), 0.37
    e, eb = synth.random_field(n, n + m), synth.random_field(m, n + m + 1)
    got = to_np(fb.mft_forward(to_gpu(e), n_d, m, du))
    assert rel_l2(got, oracle.mft(f32(e), n_d, m, du)) <= 1.5e-6
    got = to_np(fb.mft_adjoint(to_gpu(eb), n_d, n, du))
    assert rel_l2(got, oracle.mft_adjoint(f32(eb), n_d, n, du)) <= 1.5e-6


# whole 64-pair stages leave the last slices of a split without a pair (sixteen slices of 128 pairs
# over 1100 or 1300 pairs)
@pytest.mark.parametrize("n", [2200, 2600])
def test_slices_without_pairs(n):
    banner(f"folded mft {n} -> 96, empty slices")
    n_d, m, du = 0.4 * n, 96, 0.37
    e = synth.random_field(n, n)
    got = to_np(fb.mft_forward(to_gpu(e), n_d, m, du))
    assert rel_l2(got, oracle.mft(f32(e), n_d, m, du)) <= 1.5e-6


def test_rounding_errors_do_not_gather_on_the_axis():
    # Rounding errors are independent from output to output, so the rms of one row's 64 errors is
    # within 1 / sqrt(128) of any other row's, one standard deviation: a factor of 2 is eleven. The
    # sum of a matrix product that rounds with a bias puts that bias of all 4095 rows on the axis.
    n, m, n_d, du = 4095, 64, 0.4 * 4095, 0.11
    banner("mft 4095 -> 64, errors on the axis")
    rng = np.random.default_rng(7)
    e = np.exp(2j * np.pi * rng.random((n, n))) * 10.0 ** (-12.0 * rng.random((n, n)))
    d = to_np(fb.mft_forward(to_gpu(e), n_d, m, du)) - oracle.mft(f32(e), n_d, m, du)
    rows, cols = (np.sqrt(np.mean(np.abs(d) ** 2, axis=a)) for a in (1, 0))
    assert rows[m // 2] <= 2.0 * np.median(rows) and cols[m // 2] <= 2.0 * np.median(cols)


@pytest.mark.parametrize("m,n", [(256, 4096), (255, 1500), (300, 2048), (512, 700)])
def test_peaked_fields_keep_their_peak(m, n):
    # a focal field falling off as 1 / r^2 from a point off the axis. Largest error over the largest
    # result: the rounding of the intermediate product and of the result (2^-24 each), of the matrix
    # entries along both axes (2^-25 each) and of the sums, which may add as much again: 4 x 2^-24
    banner(f"mft_adjoint {m} -> {n}, peaked field")
    n_d, du = 0.4 * n, 0.37 if n < 1000 else 0.11
    rng = np.random.default_rng(m + n)
    x = np.arange(m) - m // 2
    r2 = (x[:, None] + 0.13 * m) ** 2 + (x[None, :] - 0.17 * m) ** 2
    eb = np.exp(1j * rng.normal(size=(m, m))) / (1.0 + r2 / 9.0)
    got, ref = to_np(fb.mft_adjoint(to_gpu(eb), n_d, n, du)), oracle.mft_adjoint(f32(eb), n_d, n, du)
    assert np.max(np.abs(got - ref)) <= 4 * 2.0 ** -24 * np.max(np.abs(ref))


# a large and a small output of either kernel: sums over all pairs, and short sums of a large output
@pytest.mark.parametrize("n,m", [(333, 77), (1030, 256), (2050, 65)])
@pytest.mark.parametrize("scale", [1e-36, 1e-34, 1e-30, 1e30, 1e35])
def test_float32_range(n, m, scale):
    # the bar of the products at ordinary magnitudes (test_folded_products_at_tile_edges) holds as long
    # as the results are ordinary float32 numbers
    banner(f"mft {n} <-> {m} of fields about {scale:g}")
    n_d, du = 0.4 * n, 0.11
    e, eb = scale * synth.random_field(n, n + m), scale * synth.random_field(m, n + m + 1)
    got, ref = to_np(fb.mft_forward(to_gpu(e), n_d, m, du)) / scale, oracle.mft(f32(e) / scale, n_d, m, du)
    assert rel_l2(got, ref) <= 1.5e-6
    got, ref = to_np(fb.mft_adjoint(to_gpu(eb), n_d, n, du)) / scale, oracle.mft_adjoint(f32(eb) / scale, n_d, n, du)
    assert rel_l2(got, ref) <= 1.5e-6


@pytest.mark.parametrize("n,m", [(333, 77), (1030, 256), (2050, 65)])
def test_float32_range_at_its_upper_end(n, m):
    # one value that rounds to an infinite bfloat16, and two whose difference is infinite in float32
    # while the sums they enter are not: their sine stays below sin(0.55)
    banner(f"mft {n} <-> {m} of fields at the end of float32's range")
    big, off = float(np.float32(3.398e38)), 4
    n_d = 1.2 * n
    du = 0.55 / (2 * np.pi * off * (n // 2)) * n_d
    for size, run, ref in ((n, lambda t: fb.mft_forward(t, n_d, m, du), lambda e: oracle.mft(e, n_d, m, du)),
                           (m, lambda t: fb.mft_adjoint(t, n_d, n, du), lambda e: oracle.mft_adjoint(e, n_d, n, du))):
        e = np.zeros((size, size), dtype=np.complex64)
        e[size // 2 + 1, size // 2 - off] = big
        got, want = to_np(run(to_gpu(e))), ref(e.astype(np.complex128))
        assert rel_l2(got / big, want / big) <= 1.5e-6
        e[:] = 0
        e[size // 2, size // 2 - off], e[size // 2, size // 2 + off] = -2.5e38, 2.5e38
        got, want = to_np(run(to_gpu(e))), ref(e.astype(np.complex128))
        assert rel_l2(got / big, want / big) <= 1.5e-6


# products of at most 16 pairs with a small output: no pair to 16, the two kernels' last lengths and the
# next, odd and even; outputs without a positive index, around a wave's 64 outputs (rows) and columns, a
# block's 4 rows and 32 outputs, and enough of them for eight outputs a wave
@pytest.mark.parametrize("m", [1, 2, 3, 16, 17, 18, 32, 33, 34])
@pytest.mark.parametrize("n", [1, 2, 31, 63, 66, 127, 130, 1025])
def test_products_of_few_pairs(n, m):
    # the bar of test_folded_products_at_tile_edges: fewer roundings than there
    n_d, du = max(1.0, 0.4 * n), 0.37
    eb, e = synth.random_field(m, n + m), synth.random_field(m, n + m + 1)
    got = to_np(fb.mft_adjoint(to_gpu(eb), n_d, n, du))
    assert rel_l2(got, oracle.mft_adjoint(f32(eb), n_d, n, du)) <= 1.5e-6
    got = to_np(fb.mft_forward(to_gpu(e), n_d, n, du))
    assert rel_l2(got, oracle.mft(f32(e), n_d, n, du)) <= 1.5e-6


@pytest.mark.parametrize("m", [16, 33])
def test_few_pairs_with_mask_background_and_range(m):
    # the epilogue of the products of few pairs into a window, and fields at both ends of float32's range
    n, nd, du = 300, 130, 0.37
    plane, eb, lyot = synth.random_field(n, 13), synth.random_field(m, 14), synth.lyot_stop(nd, 0.9)
    off = (n - nd) // 2
    t = to_gpu(plane)
    fb.mft_adjoint(to_gpu(eb), float(nd), nd, du, alpha=-1.0, beta=1.0, mask=to_gpu(lyot, torch.float32),
                   out=t[off:off + nd, off:off + nd])
    want = f32(plane).copy()
    want[off:off + nd, off:off + nd] = lyot * (want[off:off + nd, off:off + nd]
                                               - oracle.mft_adjoint(f32(eb), float(nd), nd, du))
    assert rel_l2(to_np(t), want) <= 1.5e-6
    for scale in (1e-35, 1e35):
        got = to_np(fb.mft_adjoint(to_gpu(scale * eb), float(nd), nd, du)) / scale
        assert rel_l2(got, oracle.mft_adjoint(f32(scale * eb) / scale, float(nd), nd, du)) <= 1.5e-6


GENERAL, SHORT, FEW = 0, 1, 2


def _kernel(f, p, q):
    return fb.lib()._ZN2fr9fold_kindEiii(f, p, q)


# the short sums' kernel along columns: inputs of one stage and of two, whole stages, one pair more and
# less, odd and even; outputs of whole tiles and ragged, odd and even
@pytest.mark.parametrize("m,n", [(33, 1999), (64, 2050), (65, 2047), (127, 2048), (128, 1780), (129, 1777), (130, 1601),
                                 (192, 1600), (255, 1601), (256, 1500), (257, 1500)])
def test_short_sums_of_large_outputs(m, n):
    # the bar of test_folded_products_at_tile_edges
    assert _kernel(n, n, m) == SHORT and _kernel(n, n, 258) == GENERAL
    banner(f"mft_adjoint {m} -> {n}, short sums")
    n_d, du = 0.4 * n, 0.37
    eb = synth.random_field(m, n + m)
    got = to_np(fb.mft_adjoint(to_gpu(eb), n_d, n, du))
    assert rel_l2(got, oracle.mft_adjoint(f32(eb), n_d, n, du)) <= 1.5e-6


@pytest.mark.parametrize("m", [65, 255])
def test_short_sums_with_mask_and_background(m):
    n, nd, du = 1700, 1555, 0.37
    assert _kernel(nd, nd, m) == SHORT
    plane, eb, lyot = synth.random_field(n, 13), synth.random_field(m, 14), synth.lyot_stop(nd, 0.9)
    off = (n - nd) // 2
    t = to_gpu(plane)
    fb.mft_adjoint(to_gpu(eb), float(nd), nd, du, alpha=-1.0, beta=1.0, mask=to_gpu(lyot, torch.float32),
                   out=t[off:off + nd, off:off + nd])
    want = f32(plane).copy()
    want[off:off + nd, off:off + nd] = lyot * (want[off:off + nd, off:off + nd]
                                               - oracle.mft_adjoint(f32(eb), float(nd), nd, du))
    assert rel_l2(to_np(t), want) <= 1.5e-6


@pytest.mark.parametrize("m,n", [(254, 8192), (255, 8191)])
def test_short_sums_along_rows(m, n):
    # rows of 255 samples on 8191 outputs, then columns of as many; every 97th row and column of the result
    assert _kernel(m, n, m) == SHORT and _kernel(n, n, m) == SHORT
    banner(f"mft_adjoint {m} -> {n}, short sums along rows")
    n_d, du = 0.4 * n, 0.37
    eb = synth.random_field(m, n + m)
    got = to_np(fb.mft_adjoint(to_gpu(eb), n_d, n, du)[::97, ::97].contiguous())
    w = oracle.mft_matrix(m, n, n_d, du)[:, ::97].conj()
    assert rel_l2(got, (du / n_d) * w.T @ f32(eb) @ w) <= 1.5e-6


@pytest.mark.parametrize("n,m", [(70, 40), (131, 60)])
def test_rows_past_32_bit_offsets(n, m):
    # a window of a plane whose 32 rows span more than 2^31 bytes: every stage element by element
    ld = (1 << 31) // (8 * 31) + 1
    assert _kernel(n, m, n) == GENERAL and 31 * ld * 8 >= 1 << 31
    banner(f"mft_forward {n} -> {m}, rows {ld} elements apart")
    n_d, du = 0.4 * n, 0.37
    e = synth.random_field(n, n + m)
    view = torch.empty((n - 1) * ld + n, dtype=torch.complex64, device="cuda:0").as_strided((n, n), (ld, 1))
    view.copy_(to_gpu(e))
    got = to_np(fb.mft_forward(view, n_d, m, du))
    assert rel_l2(got, oracle.mft(f32(e), n_d, m, du)) <= 1.5e-6
