"""GPU parity of GBS_CACHED, the conventional accelerated method (Sec. 2.2):
per-isochromat combined transitions (Eq. 7) composed at the first occurrence
of a with-RF waveform and reused from the cache, and with-ADC subsequences
evaluated at every sample from the block-start state (Eq. 4, 5, 6).

Same bar as the other modes against the FP64 oracle: max |dM| <= 1e-5 and
relative signal error <= 1e-4.
"""
import numpy as np
import pytest

import oracle
import synth
from synth import SeqBuilder
from tests.test_gpu_parity import DM_TOL, SIG_TOL, check_case, errors, run_gpu, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_03960_amd as gb
    return gb


def test_cached_gre_4096(gb):
    ph, seq = synth.workload("gre")
    check_case(gb, "gre", ph, seq, modes=("cached",))
    _, _, st = run_gpu(gb, ph, seq, gb.GBS_CACHED)
    # 32 excitations of one waveform: composed once, read from the cache 31 times
    assert (st["n_rf_cached"], st["n_distinct_rf"], st["n_adc_direct"], st["n_fallback"]) == (32, 1, 32, 0), st
    assert st["cache_bytes"] == 48 * ph.K


def test_cached_fse_small(gb):
    ph, seq = synth.workload("fse-small")
    check_case(gb, "fse-small", ph, seq, modes=("cached",))


def test_cached_epi_small(gb):
    ph, seq = synth.workload("epi-small")
    check_case(gb, "epi-small", ph, seq, modes=("cached",))


def test_cached_ragged_k_and_initial_state(gb):
    ph = synth.gre_phantom(33, 31, 3, seed=21)  # K = 3069: not a multiple of a workgroup
    seq = synth.gre_sequence(n_lines=3, n_read=24, dwell_steps=4, rf_steps=600, te=2.5e-3, tr=7e-3)
    rng = np.random.default_rng(2)
    check_case(gb, "ragged+m_init", ph, seq, modes=("cached",), m_init=rng.uniform(-0.5, 0.5, (3, ph.K)))


def test_cached_classification_paths(gb):
    """Gx/Gy/no-grads and mixed-gradient RF (all cached per isochromat),
    Gy/Gz readouts with ramps (direct), ADC with RF (stepped)."""
    from tests.test_oracle_pins import _mini_sequences
    ph = synth.tiny_phantom(nx=9, ny=7, nz=3, n_classes=3, df_levels=3)
    for seq in _mini_sequences():
        check_case(gb, f"mini:{seq.name}", ph, seq, modes=("cached",))


def test_cached_edge_cases(gb):
    ph1 = synth.gre_phantom(1, 1, 1, seed=4)  # K = 1
    seq = synth.gre_sequence(n_lines=2, n_read=8, dwell_steps=2, rf_steps=200, te=1.5e-3, tr=4e-3)
    check_case(gb, "K=1", ph1, seq, modes=("cached",))
    ph = synth.tiny_phantom(nx=6, ny=5, nz=2)
    rng = np.random.default_rng(8)
    m_init = rng.uniform(-0.5, 0.5, (3, ph.K))
    sb = SeqBuilder(1e-6, "relax-only")
    sb.relax(2e-3, (1e-5, -2e-5, 3e-6))
    check_case(gb, "relax-only", ph, sb.build(), modes=("cached",), m_init=np.full((3, ph.K), 0.3))
    # a readout before any RF reads the initial state; 700 samples take three
    # launches; one sample per launch-chunk tail; a readout without samples
    sb = SeqBuilder(1e-6, "adc-first")
    sb.adc(800, (0.004, -0.002, 0.001), np.arange(0, 700))
    sb.relax(3e-4, (1e-6, 0, 0))
    sb.adc(30, (0.0, 0.0, 0.01), [])
    sb.rf(synth.sinc_pulse(80, 1e-6, 0.7), (0, 0, 0.01))
    sb.adc(40, (0.01, 0, 0), [3])
    check_case(gb, "adc-first", ph, sb.build(), modes=("cached",), m_init=m_init)
    sb = SeqBuilder(1e-6, "b1zero")
    sb.rf(np.zeros(50), (0, 0, 0.01))
    sb.rf(synth.sinc_pulse(80, 1e-6, 0.7), (0, 0, 0.01))
    sb.adc(16, (0.01, 0, 0), np.arange(0, 17, 4))
    check_case(gb, "b1zero", ph, sb.build(), modes=("cached",))
    check_case(gb, "empty", ph, SeqBuilder(1e-6, "empty").build(), modes=("cached",), m_init=m_init)


def test_cached_infinite_relaxation_times(gb):
    ph = synth.tiny_phantom(nx=5, ny=4, nz=2, n_classes=2)
    ph.t1[::3] = np.inf
    ph.t2[1::4] = np.inf
    seq = synth.gre_sequence(n_lines=2, n_read=8, dwell_steps=2, rf_steps=200, te=1.5e-3, tr=4e-3)
    check_case(gb, "T=inf", ph, seq, modes=("cached", "plain"))


def test_cached_reuse_matches_compose_and_repeats(gb):
    """Five occurrences of one waveform (composed once, applied four times from
    the FP32 cache) against the oracle; a second call on the same context
    recomposes and gives the same bits."""
    import torch
    ph = synth.tiny_phantom(nx=8, ny=6, nz=3, n_classes=3, df_levels=3)
    sb = SeqBuilder(1e-6, "reuse")
    b1 = synth.sinc_pulse(120, 1e-6, 0.9)
    for i in range(5):
        sb.rf(b1, (0, 0, 0.01))
        sb.relax(4e-4, (2e-6 * (i + 1), -1e-6, 0))
        sb.adc(24, (0.008, 0, 0), 3 * np.arange(8))
    seq = sb.build()
    check_case(gb, "reuse", ph, seq, modes=("cached",))
    sim = gb.Simulator(0)
    sim.set_phantom(ph)
    sim.set_sequence(seq)
    M1, s1, st = sim.simulate(gb.GBS_CACHED, stats=True, flags=gb.GBS_PROFILE)
    M1, s1 = M1.cpu().numpy().copy(), s1.cpu().numpy().copy()
    M2, s2 = sim.simulate(gb.GBS_CACHED)
    torch.cuda.synchronize()
    assert np.array_equal(M1, M2.cpu().numpy()) and np.array_equal(s1, s2.cpu().numpy())
    assert (st["n_rf_cached"], st["n_distinct_rf"], st["n_adc_direct"]) == (5, 1, 5), st
    assert st["ms_compose"] > 0 and st["ms_apply"] > 0 and st["ms_adc_direct"] > 0, st
    sim.close()


def test_cached_agrees_with_grouped_and_plain(gb):
    """Three implementations of the same discrete model on one mid-size case."""
    ph, seq = synth.workload("fse-small")
    Mc, sc, _ = run_gpu(gb, ph, seq, gb.GBS_CACHED)
    Mg, sg, _ = run_gpu(gb, ph, seq, gb.GBS_GROUPED)
    Mp, sp, _ = run_gpu(gb, ph, seq, gb.GBS_PLAIN)
    for name, M, s in (("grouped", Mg, sg), ("plain", Mp, sp)):
        dm, rel = errors(Mc, sc, M, s)
        say(f"[gpu] cached vs {name}: max|dM|={dm:.3e} rel_sig={rel:.3e}")
        assert dm <= DM_TOL and rel <= SIG_TOL


@pytest.mark.parametrize("n_read,k,coils", [
    (47, 40, 1), (48, 1, 1), (48, 31, 1), (49, 32, 2), (127, 33, 1), (128, 127, 1), (129, 128, 3), (255, 129, 1),
    (256, 640, 1), (300, 65, 8),
])
def test_cached_readout_products(gb, n_read, k, coils):
    """Arithmetic readouts as matrix products: samples and isochromats around
    the edges of the tiles and chunks, all three gradients, from an initial
    state and after a transition; per readout and coil."""
    import torch
    rng = np.random.default_rng(n_read + k)
    ph = synth.gre_phantom(k, 1, 1, seed=k)
    ph.y, ph.z = (rng.uniform(-0.05, 0.05, k).astype(np.float32) for _ in range(2))
    ph.m0 = rng.uniform(0.2, 1.0, k).astype(np.float32)
    sb = SeqBuilder(1e-6, "products")
    sb.adc(2 * n_read, (3e-3, -2e-3, 1e-3), 2 * np.arange(n_read) + 1)
    sb.rf(synth.sinc_pulse(60, 1e-6, 0.9), (0, 0, 0.01))
    sb.relax(1e-3, (-1e-8, 2e-8, 0.0))
    sb.adc(3 * n_read, (0.0, 1e-3, 0.0), 3 * np.arange(n_read))
    seq = sb.build()
    m_init = rng.uniform(-0.5, 0.5, (3, k)).astype(np.float32)
    sens = (rng.uniform(0.5, 1.0, (coils, k)) * np.exp(1j * rng.uniform(-3, 3, (coils, k)))).astype(np.complex64)
    if coils > 1:
        Mr, sr = oracle.simulate_coils(ph, seq, sens, m_init=m_init)
    else:
        Mr, sr = oracle.simulate(ph, seq, m_init=m_init)
    sim = gb.Simulator(0)
    sim.set_phantom(ph)
    sim.set_sequence(seq)
    if coils > 1:
        sim.set_coils(sens)
    M, s = sim.simulate(gb.GBS_CACHED, m_init=torch.from_numpy(m_init))
    torch.cuda.synchronize()
    a, b = s.cpu().numpy().reshape(-1, n_read), np.asarray(sr).reshape(-1, n_read)
    rel = np.linalg.norm(a - b, axis=1) / np.linalg.norm(b, axis=1)
    dm = float(np.max(np.abs(M.cpu().numpy() - Mr)))
    sim.close()
    say(f"[gpu] cached products: n={n_read} K={k} P={coils} max|dM|={dm:.2e} rel {rel.max():.2e}")
    assert dm <= DM_TOL and rel.max() <= SIG_TOL


@pytest.mark.parametrize("n", [1, 2, 3, 8, 63, 64, 65, 400, 401])
@pytest.mark.parametrize("form", ["x", "y", "phase", "ramped", "two lobes", "shifted", "chirp", "short T"])
def test_symmetric_pulses(gb, n, form):
    """Transitions from half the steps (pulses symmetric in time with one B1
    phase) and from all of them, one pulse from a random state, cached and
    grouped (Gz alone, and Gx with Gz).  Bars: the FP64 transition acts on the
    FP64 state in the cached mode, so M errs by its FP32 output, 6e-8 of 1; the
    grouped mode rounds the transition's entries to FP32 (four terms, 2.4e-7)."""
    import torch
    rng = np.random.default_rng(n)
    k = 300
    ph = synth.gre_phantom(15, 5, 4, seed=n)
    ph.m0 = rng.uniform(0.2, 1.0, k).astype(np.float32)
    ph.t1[7] = ph.t2[7] = np.inf
    if form == "short T":  # a raster step and less: the second half cannot come from the first
        ph.t1[::3] = 5e-7
        ph.t2[::3] = 3e-7
    rf = synth.sinc_pulse(n, 1e-6, np.deg2rad(110.0))
    gz = np.full(n, 0.02)
    if form == "y":
        rf = synth.sinc_pulse(n, 1e-6, np.deg2rad(110.0), phase=np.pi / 2)
    elif form == "phase":
        rf = rf * np.exp(1.1j)
    elif form == "ramped":
        gz = 0.02 * np.minimum(1.0, np.minimum(np.arange(n) + 1, np.arange(n, 0, -1)) / 10.0)
    elif form == "two lobes":
        rf = rf * np.cos(np.linspace(-3, 3, n)) if n > 1 else rf
    elif form == "shifted":
        rf = np.roll(rf, 1)
    elif form == "chirp":
        rf = rf * np.exp(1j * np.linspace(-1, 1, n) ** 2)
    m_init = rng.uniform(-0.55, 0.55, (3, k)).astype(np.float32)
    for g in ((0.0, 0.0, gz), (0.3 * gz, 0.0, gz)):
        sb = SeqBuilder(1e-6, form)
        sb.rf(rf, g)
        seq = sb.build()
        Mr, _ = oracle.simulate(ph, seq, m_init=m_init)
        for mode, bar in ((gb.GBS_CACHED, 2e-7), (gb.GBS_GROUPED, 6e-7)):
            sim = gb.Simulator(0)
            sim.set_phantom(ph)
            sim.set_sequence(seq)
            sim.build_groups()
            M, _ = sim.simulate(mode, m_init=torch.from_numpy(m_init))
            torch.cuda.synchronize()
            dm = float(np.max(np.abs(M.cpu().numpy() - Mr)))
            sim.close()
            say(f"[gpu] pulse {form} n={n} mode={mode}: max|dM|={dm:.2e}")
            assert dm <= bar, (form, n, mode, dm)
