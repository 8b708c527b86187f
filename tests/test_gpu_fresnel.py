"""GPU parity of fresnel_step / fresnel_step_batched against the FP64 oracle and closed forms.

Bar (stated in the task and derived for the field): intensity relative L2 <= 1e-5; the complex
field relative L2 <= 1e-5 as well (float32 FFT error grows ~ log2 n * 6e-8)."""

import math

import numpy as np
import pytest
import torch

import oracle
from paper_1806_06467_amd import fresnel as fb
from paper_1806_06467_amd import synth
from tests.gpu_common import banner, f32, grid_plane_wave_sum, rel_l2, to_gpu, to_np

pytestmark = pytest.mark.gpu

TOL = 1e-5


def _case(n, seed):
    rng = np.random.default_rng(seed)
    field = synth.random_field(n, seed)
    amp = rng.uniform(0.3, 1.0, (n, n))
    opd = rng.normal(0.0, 60e-9, (n, n))
    lam = 550e-9 + 10e-9 * (seed % 5)
    dx = 2.0e-5
    z = 0.7 * n * dx * dx / lam          # inside the AS sampling limit
    f = 3.0 * n * dx * dx / lam          # a weak lens
    return field, amp, opd, dx, lam, z, f


def _run_gpu(field, amp, opd, dx, lam, z, f, adjoint):
    t = to_gpu(field)
    st = fb.fresnel_step(t, dx, lam, z, amp=to_gpu(amp, torch.float32), opd=to_gpu(opd, torch.float32),
                         lens_focal=f, adjoint=adjoint)
    assert st >= 0
    return to_np(t)


@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("n", [64, 128, 256, 512, 1024, 2048])
def test_fresnel_step_matches_oracle(n, adjoint):
    banner(f"fresnel_step n={n} adjoint={adjoint}")
    field, amp, opd, dx, lam, z, f = _case(n, n + adjoint)
    got = _run_gpu(field, amp, opd, dx, lam, z, f, adjoint)
    ref = oracle.fresnel_step(f32(field), dx, lam, z, amp=f32(amp), opd=f32(opd), lens_focal=f,
                              adjoint=adjoint)
    assert rel_l2(got, ref) <= TOL
    assert rel_l2(np.abs(got) ** 2, np.abs(ref) ** 2) <= TOL


@pytest.mark.parametrize("adjoint", [False, True])
def test_fresnel_step_4096_matches_oracle(adjoint):
    n = 4096
    banner(f"fresnel_step n={n} adjoint={adjoint} (oracle takes a few seconds)")
    field, amp, opd, dx, lam, z, f = _case(n, 7 + adjoint)
    got = _run_gpu(field, amp, opd, dx, lam, z, f, adjoint)
    ref = oracle.fresnel_step(f32(field), dx, lam, z, amp=f32(amp), opd=f32(opd), lens_focal=f,
                              adjoint=adjoint)
    assert rel_l2(got, ref) <= TOL
    assert rel_l2(np.abs(got) ** 2, np.abs(ref) ** 2) <= TOL


@pytest.mark.parametrize("n", [512, 4096, 8192])
def test_gaussian_beam_closed_form_full_size(n):
    banner(f"gaussian closed form n={n}")
    dx, lam, w0px = 1e-5, 550e-9, 12.0 * n / 512
    w0 = w0px * dx
    zr = math.pi * w0 * w0 / lam
    t = to_gpu(synth.gaussian_beam(n, w0px))
    fb.fresnel_step(t, dx, lam, 1.5 * zr)
    got = to_np(t)
    zeta = 1.5
    r2 = (synth.radius_grid(n) * dx) ** 2
    ref = np.exp(-r2 / (w0 * w0 * (1 + 1j * zeta))) / (1 + 1j * zeta)
    assert rel_l2(got, ref) <= TOL


@pytest.mark.parametrize("n", [2048, 8192])
def test_talbot_closed_form(n):
    banner(f"talbot n={n}")
    dx, lam, period, amp = 0.04 / 256, 0.5e-6, 2e-3, 5e-9
    opd = synth.sine_opd(n, dx, period, amp)
    t = torch.ones((n, n), dtype=torch.complex64, device="cuda:0")
    fb.fresnel_step(t, dx, lam, 4.0, opd=to_gpu(opd, torch.float32))
    got = to_np(t)
    a = 2 * math.pi * amp / lam
    theta = 2 * math.pi * ((np.arange(n) - n // 2) * dx) / period
    ref = np.broadcast_to(np.cos(a * np.sin(theta)) + np.sin(a * np.sin(theta)), (n, n))
    assert rel_l2(got, ref) <= TOL
    assert np.max(np.abs(got.imag)) <= 1e-5


@pytest.mark.parametrize("fraction", [0.05, 0.25])
def test_talbot_appendix_a_with_aperture(fraction):
    """The Talbot example of Sec. 1.1 / Fig. 1 as Appendix A prescribes it: a 2 cm radius circular
    aperture sampled by 256 px, oversampled 8x to a 2048^2 grid, a 5 nm sine OPD of 500
    cycles per metre, 0.5 um, propagated 0.05 and 0.25 Talbot lengths (Z_T = 2 p^2 / lambda =
    16 m; tests/golden/talbot_appendix_a.json), against the FP64 oracle on the whole plane. The
    conversion of phase into amplitude error: inside half the radius (away from the edge's
    ringing) the intensity's component along sin(2 pi x / p) is, as for the unbounded grating
    whose harmonic n advances by exp(-2 pi i n^2 z / Z_T), 4 J0(a) J1(a) sin(2 pi z / Z_T) to
    first order in a = 2 pi 5 nm / lambda: complete at 0.25 Z_T, 31 % of it at 0.05 Z_T."""
    n, dx, lam, period, amp_m = 2048, 0.04 / 256, 0.5e-6, 2e-3, 5e-9
    z_t = 2 * period ** 2 / lam
    z = fraction * z_t
    banner(f"talbot with aperture: 2048^2, z = {fraction} Z_T = {z} m")
    aperture = synth.circular_aperture(n, 128.0)
    opd = synth.sine_opd(n, dx, period, amp_m)
    t = torch.ones((n, n), dtype=torch.complex64, device="cuda:0")
    st = fb.fresnel_step(t, dx, lam, z, amp=to_gpu(aperture, torch.float32), opd=to_gpu(opd, torch.float32))
    assert st == 0
    got = to_np(t)
    ref = oracle.fresnel_step(np.ones((n, n), dtype=np.complex128), dx, lam, z, amp=f32(aperture), opd=f32(opd))
    assert rel_l2(got, ref) <= TOL
    from scipy.special import j0, j1
    inner = synth.radius_grid(n) < 64.0
    sin_x = np.broadcast_to(np.sin(2 * math.pi * (np.arange(n) - n // 2) * dx / period), (n, n))[inner]
    inten = np.abs(got[inner]) ** 2
    c = np.sum((inten - inten.mean()) * sin_x) / np.sum(sin_x ** 2)
    a = 2 * math.pi * amp_m / lam
    want = 4 * j0(a) * j1(a) * math.sin(2 * math.pi * fraction)
    assert abs(c - want) <= 0.01 * want


def test_round_trip_and_zero_distance_4096():
    n = 4096
    banner("round trip n=4096")
    field = synth.random_field(n, 3)
    t = to_gpu(field)
    fb.fresnel_step(t, 2e-5, 600e-9, 1.1)
    fb.fresnel_step(t, 2e-5, 600e-9, -1.1)
    assert rel_l2(to_np(t), field) <= TOL
    t = to_gpu(field)
    fb.fresnel_step(t, 2e-5, 600e-9, 0.0)
    assert rel_l2(to_np(t), field) <= TOL


def test_batched_equals_single_and_is_deterministic():
    n = 1024
    banner("batched vs single n=1024")
    lams = [500e-9, 550e-9, 600e-9]
    fields = [synth.random_field(n, 20 + i) for i in range(3)]
    rng = np.random.default_rng(5)
    opd = to_gpu(rng.normal(0, 30e-9, (n, n)), torch.float32)
    singles = []
    for i, fld in enumerate(fields):
        t = to_gpu(fld)
        fb.fresnel_step(t, 3e-5, lams[i], 0.5, opd=opd, adjoint=(i == 1))
        singles.append(to_np(t))
    ts = [to_gpu(f) for f in fields]
    fb.fresnel_step_batched(ts, 3e-5, lams, 0.5, opds=opd, adjoints=[False, True, False])
    for i in range(3):
        assert np.array_equal(to_np(ts[i]), singles[i])


@pytest.mark.parametrize("n,count", [(256, 6), (4096, 4), (3840, 3)])
def test_batched_graph_replays_equal_eager(n, count):
    """The recorded batched call (fresnel_step_batched_graph), replayed three times with new field
    contents written in place and unrelated eager work in between, equals the eager batched call
    bit for bit on every replay (forward and adjoint planes, amplitude and OPD maps); 3840 takes
    the mixed-radix sweeps."""
    banner(f"batched graph replays n={n} count={count}")
    rng = np.random.default_rng(n + count)
    amp = to_gpu(rng.uniform(0.5, 1.0, (n, n)), torch.float32)
    opd = to_gpu(rng.normal(0, 30e-9, (n, n)), torch.float32)
    lams = [500e-9 + 20e-9 * i for i in range(count)]
    adj = [i % 2 == 1 for i in range(count)]
    dx = 2.0 * math.sqrt(600e-9 * 0.5 / n)
    ts = [torch.empty((n, n), dtype=torch.complex64, device="cuda:0") for _ in range(count)]
    for rep in range(4):
        inputs = [to_gpu(synth.random_field(n, 100 * rep + i)) for i in range(count)]
        refs = [x.clone() for x in inputs]
        fb.fresnel_step_batched(refs, dx, lams, 0.5, amps=amp, opds=opd, adjoints=adj)
        for t, x in zip(ts, inputs):
            t.copy_(x)
        fb.fresnel_step_batched(ts, dx, lams, 0.5, amps=amp, opds=opd, adjoints=adj, graph=True)
        junk = torch.randn(1 << 20, device="cuda:0").sum()
        torch.cuda.synchronize()
        for i in range(count):
            assert torch.equal(ts[i], refs[i]), (rep, i)
        assert torch.isfinite(junk)


def test_warning_bit_for_undersampled_distance():
    n = 256
    t = to_gpu(synth.random_field(n, 1))
    st = fb.fresnel_step(t, 1e-5, 500e-9, 2.0 * n * 1e-10 / 500e-9)
    assert st & fb.FR_W_AS_UNDERSAMPLED


# ---- edges that are not powers of two (mixed-radix sweeps) ---------------------------------

@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("n", [6, 30, 96, 100, 210, 1000, 3000])
def test_mixed_radix_step_matches_oracle(n, adjoint):
    banner(f"fresnel_step mixed-radix n={n} adjoint={adjoint}")
    field, amp, opd, dx, lam, z, f = _case(n, 3 * n + adjoint)
    got = _run_gpu(field, amp, opd, dx, lam, z, f, adjoint)
    ref = oracle.fresnel_step(f32(field), dx, lam, z, amp=f32(amp), opd=f32(opd), lens_focal=f,
                              adjoint=adjoint)
    assert rel_l2(got, ref) <= TOL
    assert rel_l2(np.abs(got) ** 2, np.abs(ref) ** 2) <= TOL


# the padded per-wavelength grids of the broadband workload (radix plans 16.16.14, 16.15.15,
# 16.16.15, 16.9.9.3, 16.7.7.5, 16.10.5.5, 16.14.9.2: the compile-time instances of the
# mixed-radix sweeps), forward and adjoint spread over the set
@pytest.mark.parametrize("n,adjoint", [(3584, False), (3600, True), (3840, False), (3888, False), (3920, True),
                                       (4000, False), (4032, True), (3840, True)])
def test_broadband_grid_step_matches_oracle(n, adjoint):
    banner(f"fresnel_step broadband grid n={n} adjoint={adjoint} (oracle takes a few seconds)")
    field, amp, opd, dx, lam, z, f = _case(n, n + adjoint)
    got = _run_gpu(field, amp, opd, dx, lam, z, f, adjoint)
    ref = oracle.fresnel_step(f32(field), dx, lam, z, amp=f32(amp), opd=f32(opd), lens_focal=f,
                              adjoint=adjoint)
    assert rel_l2(got, ref) <= TOL
    assert rel_l2(np.abs(got) ** 2, np.abs(ref) ** 2) <= TOL


def test_mixed_size_batch_matches_oracle():
    # 28 planes (more than one launch's worth) of uneven edges, forward and adjoint mixed,
    # including power-of-two edges (64, 128, 256: the two-sweep kernels, grouped per edge)
    sizes = [96, 100, 128, 210, 64, 120, 30, 256] * 3 + [6, 2, 3, 240]
    banner(f"mixed-size batch of {len(sizes)} planes")
    cases = [_case(n, 100 + i) for i, n in enumerate(sizes)]
    adj = [i % 3 == 1 for i in range(len(sizes))]
    ts = [to_gpu(c[0]) for c in cases]
    fb.fresnel_step_batched(ts, [c[3] for c in cases], [c[4] for c in cases], [c[5] for c in cases],
                            amps=[to_gpu(c[1], torch.float32) for c in cases],
                            opds=[to_gpu(c[2], torch.float32) for c in cases],
                            lens_focals=[c[6] for c in cases], adjoints=adj)
    for i, (field, amp, opd, dx, lam, z, f) in enumerate(cases):
        ref = oracle.fresnel_step(f32(field), dx, lam, z, amp=f32(amp), opd=f32(opd), lens_focal=f,
                                  adjoint=adj[i])
        assert rel_l2(to_np(ts[i]), ref) <= TOL, (i, sizes[i])


def test_broadband_batch_equals_single_calls():
    # one batched call over all the padded grids of a 21-wavelength band equals per-plane calls
    # bit for bit (each plane takes the kernels a single call gives it: the power-of-two sweeps
    # for 4096, the mixed-radix sweeps for the others; same arithmetic per line), and a Gaussian
    # beam through a mixed batch matches its closed form
    sizes = list(synth.padded_sizes(21))
    banner(f"broadband batch of {len(sizes)} planes: {sorted(set(sizes))}")
    lams = list(synth.wavelengths(21))
    dx = 2.5e-5
    fields = [synth.random_field(n, 40 + i) for i, n in enumerate(sizes)]
    ts = [to_gpu(f) for f in fields]
    fb.fresnel_step_batched(ts, dx, lams, 0.3)
    for i, n in enumerate(sizes):
        t = to_gpu(fields[i])
        fb.fresnel_step(t, dx, lams[i], 0.3)
        assert np.array_equal(to_np(ts[i]), to_np(t)), (i, n)
    # a Gaussian beam through a mixed batch containing 4096 matches its closed form
    n, w0px = 4096, 96.0
    w0 = w0px * dx
    zr = math.pi * w0 * w0 / lams[0]
    g = [to_gpu(synth.gaussian_beam(n, w0px)), to_gpu(synth.gaussian_beam(3600, w0px))]
    fb.fresnel_step_batched(g, dx, lams[0], 1.5 * zr)
    for t, m in zip(g, (4096, 3600)):
        r2 = (synth.radius_grid(m) * dx) ** 2
        ref = np.exp(-r2 / (w0 * w0 * (1 + 1.5j))) / (1 + 1.5j)
        assert rel_l2(to_np(t), ref) <= TOL, m


@pytest.mark.parametrize("adjoint", [False, True])
def test_fresnel_step_8192_sampled_rows(adjoint):
    # the full 8192^2 plane against the oracle on sampled output rows (the separable form of the
    # paraxial step gives single rows at O(n^2) each)
    n = 8192
    banner(f"fresnel_step n=8192 adjoint={adjoint}: sampled rows vs oracle")
    rng = np.random.default_rng(81 + adjoint)
    field = f32(synth.random_field(n, 81 + adjoint))
    amp = f32(rng.uniform(0.3, 1.0, (n, n)))
    opd = f32(rng.normal(0.0, 60e-9, (n, n)))
    dx, lam, z = 1.25e-5, 550e-9, 1.0
    t = to_gpu(field)
    fb.fresnel_step(t, dx, lam, z, amp=to_gpu(amp, torch.float32), opd=to_gpu(opd, torch.float32),
                    adjoint=adjoint)
    rows = [0, 1, 1234, n // 2, 5000, n - 1]
    torch.cuda.synchronize()
    got = t[rows].cpu().numpy().astype(np.complex128)
    ph = oracle.optic_phasor(n, dx, lam, amp=amp, opd=opd)
    if adjoint:
        ref = oracle.as_propagate_rows(field, dx, lam, -z, rows) * np.conj(ph[rows])
    else:
        ref = oracle.as_propagate_rows(field * ph, dx, lam, z, rows)
    assert rel_l2(got, ref) <= TOL


def test_autotuner_choices_keep_parity(tmp_path):
    # tune the sweeps for a power-of-two and a mixed-radix edge and the MFT GEMMs, then the
    # tuned kernels still match the oracle; the choices survive a save / load round trip and a
    # corrupted file is refused
    banner("autotune: sweeps 4096 and 3840, MFT 4096 <-> 256")
    fb.autotune_fresnel(4096)
    fb.autotune_fresnel(3840)
    fb.autotune_mft(4096, 256)
    for n, adjoint in ((3840, False), (4096, True)):
        field, amp, opd, dx, lam, z, f = _case(n, 7 * n + adjoint)
        got = _run_gpu(field, amp, opd, dx, lam, z, f, adjoint)
        ref = oracle.fresnel_step(f32(field), dx, lam, z, amp=f32(amp), opd=f32(opd), lens_focal=f,
                                  adjoint=adjoint)
        assert rel_l2(got, ref) <= TOL
    # a mixed batch uses the tuned mixed-radix order
    t1, t2 = to_gpu(synth.random_field(3840, 5)), to_gpu(synth.random_field(96, 6))
    fb.fresnel_step_batched([t1, t2], 2.5e-5, 550e-9, 0.3)
    ref = oracle.fresnel_step(f32(synth.random_field(3840, 5)), 2.5e-5, 550e-9, 0.3)
    assert rel_l2(to_np(t1), ref) <= TOL
    path = tmp_path / "tune.txt"
    fb.autotune_save(str(path))
    text = path.read_text()
    assert "sweep 4096" in text and "plan 3840" in text and "gemm 4096 256 4096" in text
    fb.autotune_load(str(path))
    bad = tmp_path / "bad.txt"
    # not a factorisation of 3840 into supported radices: 17; radix 11; product 3600; a sixth
    # radix's bits after a zero radix
    for line in ("plan 3840 17", "plan 3840 %d" % (11 | (16 << 5) | (15 << 10)),
                 "plan 3840 %d" % (15 | (16 << 5) | (15 << 10)),
                 "plan 3840 %d" % (3 | (16 << 5) | (16 << 10) | (5 << 15) | (2 << 25))):
        bad.write_text(line + "\n")
        with pytest.raises(fb.FrError):
            fb.autotune_load(str(bad))
    # another factorisation of 3840 (not an order of its greedy radices) is accepted
    good = tmp_path / "good.txt"
    good.write_text("plan 3840 %d\n" % (3 | (16 << 5) | (16 << 10) | (5 << 15)))
    fb.autotune_load(str(good))


def test_sweep_variants_4096_agree_bitwise(tmp_path):
    """The tile variants of the 4096 sweeps (rows per block, columns per tile, half-size LDS
    exchanges: instances of one kernel template) compute the same planes bit for bit, on batches
    of one to three planes of different wavelengths launched together (a tuned group of three
    planes per launch) and one plane per launch, forward and adjoint with a dense optic; variant
    0 against the oracle."""
    n = 4096
    saved = tmp_path / "saved.txt"
    fb.autotune_save(str(saved))
    rng = np.random.default_rng(4096)
    amp = rng.uniform(0.5, 1.0, (n, n))
    opd = rng.normal(0, 40e-9, (n, n))
    amp_g, opd_g = to_gpu(amp, torch.float32), to_gpu(opd, torch.float32)
    lams = [500e-9, 550e-9, 600e-9]
    dx, z = 2.5e-5, 1.0
    fields = [synth.random_field(n, 900 + i) for i in range(3)]
    results = {}
    try:
        for v in range(4):
            for group in (1, 3):
                (tmp_path / "v.txt").write_text("sweep 4096 %d %d\n" % (v, group))
                fb.autotune_load(str(tmp_path / "v.txt"))
                for adjoint in (False, True):
                    banner(f"sweep variant {v}: {group} plane(s) per launch adjoint={adjoint}")
                    ts = [to_gpu(f) for f in fields]
                    fb.fresnel_step_batched(ts, dx, lams, z, amps=amp_g, opds=opd_g, adjoints=adjoint)
                    torch.cuda.synchronize()
                    results[(v, group, adjoint)] = [t.cpu() for t in ts]
                    del ts
    finally:
        fb.autotune_load(str(saved))
    for key, planes in results.items():
        ref = results[(0, 1, key[2])]
        for i in range(3):
            assert torch.equal(planes[i], ref[i]), key
    for adjoint in (False, True):
        want = oracle.fresnel_step(f32(fields[2]), dx, lams[2], z, amp=f32(amp), opd=f32(opd), adjoint=adjoint)
        got = results[(0, 3, adjoint)][2].numpy().astype(np.complex128)
        assert rel_l2(got, want) <= TOL, adjoint


def test_tuning_change_drops_recorded_graphs(tmp_path):
    """A recorded batched call replays its recording (one graph launch) until the kernel choices
    change: loading tuned choices drops every recording, so the next call runs the sweeps eagerly
    (and records again)."""
    n = 256
    saved = tmp_path / "saved.txt"
    fb.autotune_save(str(saved))
    ts = [to_gpu(synth.random_field(n, 70 + i)) for i in range(2)]

    def launches():
        fb.profile_read()
        fb.profile_enable(True)
        fb.fresnel_step_batched(ts, 2e-5, [500e-9, 600e-9], 0.05, graph=True)
        torch.cuda.synchronize()
        fb.profile_enable(False)
        return {k.partition("/")[0] for k in fb.profile_read()}
    try:
        launches()
        assert launches() == {"fresnel_graph"}
        fb.autotune_load(str(saved))
        assert "row_sweep" in launches()
        assert launches() == {"fresnel_graph"}
    finally:
        fb.autotune_load(str(saved))


def test_table_cache_bound_is_applied_between_calls_only():
    # With the cache bound at 2 tables, a batch of five planes over five distances needs six
    # tables (five transfer functions and the FFT roots): the bound must not free any of them
    # while the call runs, and the next call (which starts over the bound) rebuilds what it
    # needs. Every plane of both calls matches the oracle.
    n, dx, lam = 256, 2e-5, 550e-9
    banner("table cache bound 2 across batched calls")
    fb.set_cache_limit(2)
    try:
        for call in range(2):
            zs = [(0.1 + 0.05 * i + 0.013 * call) * n * dx * dx / lam for i in range(5)]
            fields = [synth.random_field(n, 40 + 5 * call + i) for i in range(5)]
            ts = [to_gpu(f) for f in fields]
            fb.fresnel_step_batched(ts, dx, lam, zs)
            for i in range(5):
                ref = oracle.as_propagate(f32(fields[i]), dx, lam, zs[i])
                assert rel_l2(to_np(ts[i]), ref) <= TOL
        # single exact steps over a scan of distances (one parameter table each)
        field = synth.random_field(n, 60)
        for k in range(4):
            z = (0.2 + 0.1 * k) * n * dx * dx / lam
            t = to_gpu(field)
            fb.fresnel_step_exact(t, dx, lam, z)
            assert rel_l2(to_np(t), oracle.as_propagate_exact(f32(field), dx, lam, z)) <= TOL
    finally:
        fb.set_cache_limit(4096)


@pytest.mark.parametrize("adjoint", [False, True])
def test_fresnel_step_8192_plane_waves_closed_form(adjoint):
    """The whole 8192^2 plane against a closed form: each grid plane wave of a sum is multiplied
    by the paraxial transfer function of its frequency, exp(-i pi lambda z f^2), formed here in
    float64 (conjugated for the adjoint); frequencies up to the Nyquist corner."""
    n, dx, lam, z = 8192, 1.25e-5, 550e-9, 1.0
    banner(f"fresnel_step n=8192 plane waves adjoint={adjoint}")
    waves = [(1, 0, 1.0), (-37, 1500, 0.6j), (4000, -2500, 0.5), (-4096, -4096, 0.25), (2048, 7, -0.4)]
    t = torch.from_numpy(grid_plane_wave_sum(n, waves, np.complex64)).to("cuda:0")
    fb.fresnel_step(t, dx, lam, z, adjoint=adjoint)
    expected = []
    for kx, ky, a in waves:
        hk = np.exp(-1j * np.pi * lam * z * (kx * kx + ky * ky) / (n * dx) ** 2)
        expected.append((kx, ky, a * (np.conj(hk) if adjoint else hk)))
    ref = grid_plane_wave_sum(n, expected)
    got = to_np(t)
    del t
    assert rel_l2(got, ref) <= TOL


def _pack(*radices):
    return sum(r << (5 * i) for i, r in enumerate(radices))


@pytest.mark.parametrize("n,default,greedy,other", [
    (3600, (15, 16, 15), (16, 15, 15), (15, 15, 16)),
    (3584, (7, 16, 16, 2), (16, 16, 14), (14, 16, 16)),
    (3840, (3, 16, 16, 5), (16, 16, 15), (15, 16, 16)),
    (4032, (9, 16, 14, 2), (16, 14, 9, 2), (2, 9, 14, 16)),
])
def test_broadband_grid_plans_match_oracle(n, default, greedy, other, tmp_path):
    """A broadband grid edge under three pass orders (a tuning file's `plan` line): its default
    (the register-resident sweeps), the greedy order (the compile-time instance) and another order
    (the runtime-planned sweeps), forward and adjoint, each against the oracle."""
    banner(f"mixed-radix n={n}: register-resident {default}, compile-time {greedy}, runtime {other}")
    field, amp, opd, dx, lam, z, f = _case(n, 77)
    ref = oracle.fresnel_step(f32(field), dx, lam, z, amp=f32(amp), opd=f32(opd), lens_focal=f)
    ref_adj = oracle.fresnel_step(f32(field), dx, lam, z, amp=f32(amp), opd=f32(opd), lens_focal=f, adjoint=True)
    path = tmp_path / "tune.txt"
    try:
        for order in (default, greedy, other):
            path.write_text("plan %d %d\n" % (n, _pack(*order)))
            fb.autotune_load(str(path))
            assert rel_l2(_run_gpu(field, amp, opd, dx, lam, z, f, False), ref) <= TOL, order
            assert rel_l2(_run_gpu(field, amp, opd, dx, lam, z, f, True), ref_adj) <= TOL, order
    finally:
        path.write_text("plan %d %d\n" % (n, _pack(*default)))
        fb.autotune_load(str(path))


def test_context_created_with_a_tuning_file(tmp_path):
    """fr_create takes a tuning file: a valid one is applied at creation, a malformed one fails
    the call (FR_EINVAL) and leaves no context."""
    banner("fr_create with a tuning file")
    good = tmp_path / "good.txt"
    good.write_text("sweep 4096 1 0\nplan 3600 %d\n" % (16 | (15 << 5) | (15 << 10)))
    ctx = fb.Context(0, tune_file=str(good))
    assert ctx.handle
    ctx.close()
    bad = tmp_path / "bad.txt"
    bad.write_text("sweep 4096 99 0\n")
    with pytest.raises(fb.FrError) as err:
        fb.Context(0, tune_file=str(bad))
    assert err.value.status == fb.FR_EINVAL


@pytest.mark.parametrize("n,count", [(2048, 2), (2048, 3), (2048, 5), (8192, 2)])
def test_pipelined_column_tiles_per_block_agree_bitwise(n, count):
    """The pipelined column sweep walks more tiles per block the more planes share its launch (from
    one tile to sixteen); every plane of a batch is the single call's plane bit for bit."""
    banner(f"pipelined column sweep n={n}: {count} planes")
    dx, z = 2.5e-5, n / 4096.0
    lams = [500e-9 + 20e-9 * i for i in range(count)]
    g = torch.Generator(device="cuda:0").manual_seed(n + count)
    fields = [torch.randn((n, n), generator=g, device="cuda:0", dtype=torch.complex64) for _ in range(count)]
    amp = 0.5 + 0.5 * torch.rand((n, n), generator=g, device="cuda:0")
    for adjoint in (False, True):
        batch = [f.clone() for f in fields]
        fb.fresnel_step_batched(batch, dx, lams, z, amps=amp, adjoints=adjoint)
        for f, lam, got in zip(fields, lams, batch):
            one = f.clone()
            fb.fresnel_step(one, dx, lam, z, amp=amp, adjoint=adjoint)
            assert torch.equal(one, got)


@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("n", [2, 255, 256 + 14, 511 - 7, 525, 1023 - 15, 1029, 2025, 2058])
def test_mixed_radix_class_edges(n, adjoint):
    """Edges just below and above the classes of the runtime mixed-radix sweeps (256, 512, 1024,
    2048 points per line), odd ones among them, row blocks that end past the plane included."""
    if not fb.lib().fr_fft_size_supported(n):
        n = max(m for m in range(2, n) if fb.lib().fr_fft_size_supported(m))
    banner(f"mixed-radix class edge n={n} adjoint={adjoint}")
    field, amp, opd, dx, lam, z, f = _case(n, 3 * n + adjoint)
    got = _run_gpu(field, amp, opd, dx, lam, z, f, adjoint)
    ref = oracle.fresnel_step(f32(field), dx, lam, z, amp=f32(amp), opd=f32(opd), lens_focal=f, adjoint=adjoint)
    assert rel_l2(got, ref) <= TOL


@pytest.mark.parametrize("n,plan", [(3888, (18, 12, 18)), (3920, (14, 10, 28)), (4000, (20, 10, 20)),
                                    (4032, (24, 14, 12))])
def test_three_pass_plans_in_any_company(n, plan, tmp_path):
    """The three-pass register-resident plans (radices past 16, named by a tuning file) against
    the oracle's separable form on sampled columns, and bit for bit the same in a batch with edges
    of other plans."""
    banner(f"three-pass plan n={n}")
    dx, lam, z = 2.5e-5, 550e-9, 0.9
    saved = tmp_path / "saved.txt"
    fb.autotune_save(str(saved))
    (tmp_path / "plan.txt").write_text("plan %d %d\n" % (n, plan[0] | plan[1] << 5 | plan[2] << 10))
    try:
        fb.autotune_load(str(tmp_path / "plan.txt"))
        field = synth.random_field(n, n)
        one = to_gpu(field)
        fb.fresnel_step(one, dx, lam, z)
        others = [to_gpu(synth.random_field(m, m)) for m in (250, 1000, 2500)]
        batch = [others[2], to_gpu(field), others[0], to_gpu(field), others[1]]
        fb.fresnel_step_batched(batch, dx, lam, z)
        assert torch.equal(batch[1], one) and torch.equal(batch[3], one)
    finally:
        fb.autotune_load(str(saved))
    # sampled columns: the row pass of every row, then the column pass of a few columns
    k = np.fft.fftfreq(n, d=1.0 / n)
    h = np.exp(-1j * np.pi * lam * z * (k / (n * dx)) ** 2)
    rows = np.fft.ifft(np.fft.fft(f32(field), axis=1) * h, axis=1)[:, [0, 1, n // 2, n - 1]]
    want = np.fft.ifft(np.fft.fft(rows, axis=0) * h[:, None], axis=0)
    assert rel_l2(to_np(one)[:, [0, 1, n // 2, n - 1]], want) <= TOL


@pytest.mark.parametrize("n,count", [(4096, 2), (4096, 5), (8192, 2)])
def test_pipelined_column_tiles_of_shared_launches(n, count, tmp_path):
    """Large planes share a launch only when a tuning file says so (two are past the last-level cache): their
    blocks then walk 8, 16 and 32 tiles in place of 4, 4 and 16, with the single call's bits."""
    banner(f"pipelined column sweep n={n}: {count} planes in one launch")
    saved, shared = tmp_path / "saved.txt", tmp_path / "shared.txt"
    fb.autotune_save(str(saved))
    shared.write_text("sweep %d 0 %d\n" % (n, count))
    dx, lam, z = 2.5e-5, 550e-9, n / 4096.0
    g = torch.Generator(device="cuda:0").manual_seed(n + count)
    fields = [torch.randn((n, n), generator=g, device="cuda:0", dtype=torch.complex64) for _ in range(count)]
    try:
        for adjoint in (False, True):
            fb.autotune_load(str(shared))
            batch = [f.clone() for f in fields]
            fb.fresnel_step_batched(batch, dx, lam, z, adjoints=adjoint)
            shared.write_text("sweep %d 0 0\n" % n)
            fb.autotune_load(str(shared))
            for f, got in zip(fields, batch):
                one = f.clone()
                fb.fresnel_step(one, dx, lam, z, adjoint=adjoint)
                assert torch.equal(one, got)
            shared.write_text("sweep %d 0 %d\n" % (n, count))
    finally:
        shared.write_text("sweep %d 0 0\n" % n)
        fb.autotune_load(str(shared))
        fb.autotune_load(str(saved))


@pytest.mark.parametrize("edges", [(250, 270), (100, 500, 500, 1000, 1875), (255, 256, 257, 512, 520, 1029, 2025),
                                   (250, 1000, 2058, 3000), (225, 600, 3888, 3969, 4050)])
def test_mixed_edges_keep_the_single_planes_bits(edges):
    """Planes of any classes of line lengths in one call, both directions and with maps: each has the bits of
    its own call, whichever instance its launch takes."""
    edges = [n if fb.lib().fr_fft_size_supported(n) else max(m for m in range(2, n) if fb.lib().fr_fft_size_supported(m))
             for n in edges]
    banner(f"mixed edges {edges}")
    g = torch.Generator(device="cuda:0").manual_seed(sum(edges))
    fields = [torch.randn((n, n), generator=g, device="cuda:0", dtype=torch.complex64) for n in edges]
    amps = [0.5 + 0.5 * torch.rand((n, n), generator=g, device="cuda:0") for n in edges]
    opds = [5e-8 * torch.randn((n, n), generator=g, device="cuda:0") for n in edges]
    dx, lam, zs = 2.5e-5, 550e-9, [n / 4096.0 for n in edges]
    for adjoints in ([False] * len(edges), [True] * len(edges), [i % 2 == 1 for i in range(len(edges))]):
        batch = [f.clone() for f in fields]
        fb.fresnel_step_batched(batch, dx, lam, zs, amps=amps, opds=opds, lens_focals=[2.0] * len(edges), adjoints=adjoints)
        for n, f, amp, opd, z, adj, got in zip(edges, fields, amps, opds, zs, adjoints, batch):
            one = f.clone()
            fb.fresnel_step(one, dx, lam, z, amp=amp, opd=opd, lens_focal=2.0, adjoint=adj)
            assert torch.equal(one, got), n
