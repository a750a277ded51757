"""GPU parity of the per-run form of the grouped simulation: a call from
(0, 0, M0) steps every run of equal (x, z, T1, T2, dB0) once.  Against the FP64
oracle at the edges of the form: run lengths around the wavefront's chunks,
numbers of phase-encode lines around the tiles of 32 and 256, x-groups of more
runs than a wavefront holds, several coils and batches, and sequences that the
form does not take.  M0 is random per isochromat, so that every line carries
signal; bars per readout: |dM| <= 1e-5, relative signal 1e-4 (those of the
other parity tests)."""
import numpy as np
import pytest

import oracle
import synth
from synth import GAMMA_BAR, SeqBuilder

pytestmark = pytest.mark.gpu

DM_TOL = 1e-5
SIG_TOL = 1e-4


@pytest.fixture(scope="module")
def gb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_03960_amd as gb
    return gb


def phantom(nx, ny, nz, seed=3, classes=2, levels=2):
    rng = np.random.default_rng(seed)
    ph = synth.tiny_phantom(nx, ny, nz, n_classes=classes, df_levels=levels, seed=seed, fov=(0.2, 0.2, 0.01))
    ph.m0 = rng.uniform(0.1, 1.0, ph.K).astype(np.float32)
    ph.m0[rng.integers(0, ph.K, max(1, ph.K // 16))] = 0.0
    ph.t1[0] = np.inf
    return ph


def sequence(ky, n_read=4, rf_axis=(0, 0, 1), rewind=True, end_ky=0.0, keep_y=False, rf_steps=48):
    """A gradient-echo train with the given phase-encode steps (units of 1 / FOV)."""
    sb = SeqBuilder(1e-6, "lines")
    b1 = synth.sinc_pulse(rf_steps, 1e-6, np.deg2rad(50.0))
    amp = 0.02
    for i, k in enumerate(ky):
        m = k / (GAMMA_BAR * 0.2)
        sb.rf(b1 * np.exp(0.3j * (i % 7)), tuple(amp * a for a in rf_axis))
        sb.relax(1e-3, (-3e-9, m, -0.4 * amp * rf_steps * 1e-6))
        sb.adc(4 * n_read, (2e-4, 0.0, 0.0), 4 * np.arange(n_read) + 2)
        sb.relax(4e-3, (2e-9, 0.0 if keep_y else (-m if rewind or i + 1 < len(ky) else 0.0), 3e-7))
    if end_ky:
        sb.relax(2e-3, (1e-9, end_ky / (GAMMA_BAR * 0.2), 0.0))
    return sb.build()


def grouped(gb, ph, seq, sens=None, axes=None, explicit=False):
    import torch
    sim = gb.Simulator(0)
    sim.set_phantom(ph)
    sim.set_sequence(seq)
    if sens is not None:
        sim.set_coils(sens)
    sim.build_groups(gb.GBS_AX_ALL if axes is None else axes)
    mi = None
    if explicit:
        z = np.zeros_like(ph.m0)
        mi = torch.from_numpy(np.stack([z, z, ph.m0]))
    M, s = sim.simulate(gb.GBS_GROUPED, m_init=mi)
    torch.cuda.synchronize()
    out = M.cpu().numpy().astype(np.float64), s.cpu().numpy().copy()
    sim.close()
    return out


def check(gb, name, ph, seq, sens=None, axes=None):
    if sens is None:
        Mr, sr = oracle.simulate(ph, seq)
    else:
        Mr, sr = oracle.simulate_coils(ph, seq, sens)
    n_read = int(seq.n_samples.max())
    ref = np.asarray(sr).reshape(-1, n_read)
    print(f"[gpu] runs {name}: K={ph.K}", flush=True)
    M, s = grouped(gb, ph, seq, sens, axes)
    dm = float(np.max(np.abs(M - Mr)))
    rel = np.linalg.norm(s.reshape(-1, n_read) - ref, axis=1) / np.linalg.norm(ref, axis=1)
    print(f"[gpu] runs {name}: max|dM|={dm:.2e} rel per readout {rel.max():.2e}", flush=True)
    assert dm <= DM_TOL and rel.max() <= SIG_TOL, (name, dm, float(rel.max()), int(rel.argmax()))


@pytest.mark.parametrize("ny", [2, 3, 7, 8, 9, 31, 33, 63, 64, 65, 127, 129, 200])
def test_run_lengths(gb, ny):
    check(gb, f"ny={ny}", phantom(5, ny, 3, seed=ny), sequence(range(-5, 6)))


@pytest.mark.parametrize("lines", [1, 2, 31, 32, 33, 128, 129, 255, 256, 257, 513])
def test_line_counts(gb, lines):
    check(gb, f"lines={lines}", phantom(3, 41, 2, seed=lines), sequence(range(-(lines // 2), lines - lines // 2)))


@pytest.mark.parametrize("name,ky", [
    ("offset", [20.25 + 0.5 * i for i in range(37)]),
    ("descending", list(range(40, 3, -1))),
    ("gaps", [0, 3, 7, 11, 60, 61, 255]),
    ("repeated", [4, 4, -2, 4, 9, -2]),
    ("interleaved", [16 * e + s - 64 for s in range(16) for e in range(8)]),
    ("uneven", [0.0, 1.0, 2.7182, 5.1, 9.33, 11.0]),  # not on a grid: swept per isochromat
    ("wide", [0, 1, 5000]),                            # grid of more lines than the form takes
])
def test_line_grids(gb, name, ky):
    check(gb, name, phantom(4, 50, 2, seed=len(ky)), sequence(ky))


@pytest.mark.parametrize("nz", [12, 63, 64, 65, 130])
def test_groups_beyond_a_wavefront(gb, nz):
    ph = phantom(7, 9, nz, seed=nz, classes=1, levels=1)
    check(gb, f"nz={nz}", ph, sequence(range(-8, 9)))


@pytest.mark.parametrize("coils", [1, 2, 3, 4, 5, 8])
def test_coils(gb, coils):
    ph = phantom(6, 30, 3, seed=coils)
    rng = np.random.default_rng(coils)
    sens = synth.coil_maps(ph, coils) * rng.uniform(0.5, 1.5, (coils, ph.K))
    check(gb, f"coils={coils}", ph, sequence(range(-20, 20)), sens=sens.astype(np.complex64))


@pytest.mark.parametrize("name,kw,axes", [
    ("final y moment", dict(ky=range(-6, 6), rewind=False, end_ky=3.5), None),
    ("x transition", dict(ky=range(-6, 6), rf_axis=(1, 0, 0)), None),
    ("no gradient", dict(ky=range(-6, 6), rf_axis=(0, 0, 0)), None),
    ("oblique", dict(ky=range(-6, 6), rf_axis=(0.3, 0, 1)), None),
    ("without x-z groups", dict(ky=range(-6, 6)), 7),
    ("without z groups", dict(ky=range(-6, 6), rf_axis=(0, 0, 0)), 3),
    ("y transition", dict(ky=range(-6, 6), rf_axis=(0, 1, 0)), None),       # swept
    ("y moment at a transition", dict(ky=range(-6, 6), keep_y=True), None),  # swept
])
def test_forms(gb, name, kw, axes):
    check(gb, name, phantom(6, 33, 3, seed=11), sequence(**kw), axes=axes)


def test_batches_of_runs(gb):
    """More runs than one batch of Y holds (8 coils x 64 lines), against a call with
    the initial state given explicitly, which sweeps over the isochromats."""
    ph = phantom(300, 4, 120, seed=5, classes=3, levels=5)
    rng = np.random.default_rng(8)
    sens = (synth.coil_maps(ph, 8) * rng.uniform(0.5, 1.5, (8, ph.K))).astype(np.complex64)
    seq = sequence(range(-18, 18), n_read=3, rf_steps=32)
    Ma, sa = grouped(gb, ph, seq, sens)
    Mb, sb = grouped(gb, ph, seq, sens, explicit=True)
    rel = np.linalg.norm(sa - sb, axis=1) / np.linalg.norm(sb, axis=1)  # per coil
    assert np.max(np.abs(Ma - Mb)) <= DM_TOL and rel.max() <= SIG_TOL


@pytest.mark.parametrize("lines,n_read,nx", [
    (3, 5, 6),       # too few readouts of one timing: evaluated one by one
    (4, 1, 1), (4, 16, 3), (5, 17, 8), (63, 31, 9), (64, 127, 5), (65, 128, 4), (129, 129, 3),
    (6, 40, 40), (6, 40, 230),  # groups around the chunks of 32 and the splits
])
def test_readout_products(gb, lines, n_read, nx):
    """Readouts of equal timing as matrix products: rows, samples and groups
    around the edges of the tiles."""
    seq = sequence(range(-(lines // 2), lines - lines // 2), n_read=n_read)
    check(gb, f"lines={lines} read={n_read} nx={nx}", phantom(nx, 11, 2, seed=nx), seq)


def test_readouts_of_two_timings(gb):
    """Two classes of readouts, and one readout of a third timing."""
    sb = SeqBuilder(1e-6, "mixed")
    b1 = synth.sinc_pulse(40, 1e-6, np.deg2rad(40.0))
    for i in range(11):
        sb.rf(b1, (0.0, 0.0, 0.02))
        sb.relax(1e-3, (-2e-9, (i - 5) / (GAMMA_BAR * 0.2), -4e-7))
        s = 1.0 if i % 2 else -1.0
        sb.adc(40, (s * 2e-4, 0.0, 0.0), 4 * np.arange(10) + (2 if i != 7 else 1))
        sb.relax(3e-3, (1e-9, -(i - 5) / (GAMMA_BAR * 0.2), 3e-7))
    check(gb, "two timings", phantom(9, 21, 3, seed=77), sb.build())
