"""Cached readouts with receive coils at the edges of the rule that takes the
matrix product (48 samples; with coils 28 + 10 P, at most 86, from 2^17
isochromats on): the signal against GBS_PLAIN, which steps in FP64 (bars of the
other parity tests), and the time and the error of the shortest product against
one sample less, which is never one."""
import numpy as np
import pytest

import synth
from synth import SeqBuilder
from test_gpu_runs import DM_TOL, SIG_TOL, gb  # noqa: F401  (gb: fixture)

pytestmark = pytest.mark.gpu


def setup(gb, K, coils, n_read, lines=2):  # noqa: F811
    rng = np.random.default_rng(K % 1000 + coils)
    f = lambda v: np.ascontiguousarray(v, np.float32)
    ph = synth.Phantom(*(f(rng.uniform(-0.1, 0.1, K)) for _ in range(2)), f(rng.uniform(-4e-3, 4e-3, K)),
                       f(rng.uniform(0.3, 1.5, K)), f(rng.uniform(0.03, 0.2, K)), f(rng.uniform(-40, 40, K)),
                       f(rng.uniform(0.2, 1.0, K)))
    sb = SeqBuilder(1e-6, "coils")
    for _ in range(lines):
        sb.rf(synth.sinc_pulse(40, 1e-6, 0.7), (0.0, 0.0, 0.01))
        sb.relax(1e-4, (-1e-9, 2e-9, 0.0))
        sb.adc(2 * n_read, (1e-4, 2e-5, 0.0), 2 * np.arange(n_read))
    seq = sb.build()
    sens = (rng.uniform(0.5, 1.0, (coils, K)) * np.exp(1j * rng.uniform(-3, 3, (coils, K)))).astype(np.complex64)
    sim = gb.Simulator(0)
    sim.set_phantom(ph)
    sim.set_sequence(seq)
    if coils > 1:
        sim.set_coils(sens)
    return sim, seq


@pytest.mark.parametrize("K,coils,n_read", [
    (131071, 8, 48), (131072, 8, 48), (131072, 8, 85), (131073, 8, 86), (131072, 3, 57), (131072, 3, 58),
    (131072, 2, 48), (131072, 1, 48), (131072, 1, 47),
])
def test_rule(gb, K, coils, n_read):  # noqa: F811
    import torch
    sim, seq = setup(gb, K, coils, n_read)
    print(f"[gpu] cached coils K={K} P={coils} n={n_read}", flush=True)
    M, s = sim.simulate(gb.GBS_CACHED)
    Mp, sp = sim.simulate(gb.GBS_PLAIN)
    torch.cuda.synchronize()
    a, b = s.cpu().numpy().reshape(-1, n_read), sp.cpu().numpy().reshape(-1, n_read)
    rel = np.linalg.norm(a - b, axis=1) / np.linalg.norm(b, axis=1)
    dm = float((M.double() - Mp.double()).abs().max())
    sim.close()
    print(f"[gpu] cached coils K={K} P={coils} n={n_read}: max|dM|={dm:.2e} rel {rel.max():.2e}", flush=True)
    assert dm <= DM_TOL and rel.max() <= SIG_TOL


@pytest.mark.parametrize("coils", [1, 3, 4, 6, 8])
def test_one_sample_more_costs_no_more(gb, coils):  # noqa: F811
    """48 samples of 600000 isochromats take no longer than 47 and a tenth (with 8
    coils a product took 1.4 times as long)."""
    ms = []
    for n_read in (47, 48):
        sim, _ = setup(gb, 600000, coils, n_read, lines=4)
        ms.append(min(sim.simulate(gb.GBS_CACHED, flags=gb.GBS_PROFILE, stats=True)[2]["ms_adc_direct"] for _ in range(6)))
        sim.close()
    print(f"[gpu] cached readouts, {coils} coils: 47 samples {ms[0] * 250:.1f} us, 48 samples {ms[1] * 250:.1f} us", flush=True)
    assert ms[1] <= 1.1 * ms[0]


@pytest.mark.parametrize("equal", [False, True])
def test_product_errs_no_more_than_direct(gb, equal):  # noqa: F811
    """48 samples (a product) against GBS_PLAIN err by no more than 47 (evaluated
    directly) and a quarter, for random isochromats and for equal ones (whose
    roundings go one way)."""
    import torch
    K = 100000
    rng = np.random.default_rng(5)
    f = lambda v: np.ascontiguousarray(v, np.float32)
    u = (lambda a, b: np.full(K, 0.37 * a + 0.63 * b)) if equal else (lambda a, b: rng.uniform(a, b, K))
    ph = synth.Phantom(f(rng.uniform(-0.1, 0.1, K)), f(u(-0.1, 0.1)), f(u(-1e-3, 1e-3)), f(u(0.6, 1.0)), f(u(0.05, 0.09)),
                       f(u(-4, 4)), f(u(0.5, 1.0)))
    err = []
    for n_read in (47, 48):
        sb = SeqBuilder(1e-6, "errors")
        for i in range(6):
            sb.rf(synth.sinc_pulse(200, 1e-6, 0.5), (0.0, 0.0, 0.01))
            sb.relax(5e-4, (-3e-9 if i % 2 else -2e-8, 0.0, -1e-6))
            sb.adc(4 * n_read, (2e-4, 0.0, 0.0), 4 * np.arange(n_read) + 2)
            sb.relax(1e-3, (1e-9, 0.0, 0.0))
        sim = gb.Simulator(0)
        sim.set_phantom(ph)
        sim.set_sequence(sb.build())
        s = sim.simulate(gb.GBS_CACHED)[1].cpu().numpy()
        ref = sim.simulate(gb.GBS_PLAIN)[1].cpu().numpy()
        sim.close()
        err.append(float(np.linalg.norm(s - ref) / np.linalg.norm(ref)))
    print(f"[gpu] cached readouts, equal={equal}: direct errs by {err[0]:.2e}, product by {err[1]:.2e}", flush=True)
    assert err[1] <= 1.25 * err[0]


@pytest.mark.parametrize("case", ["peak 16", "peak 24", "no phase"])
def test_product_is_not_biased(gb, case):  # noqa: F811
    """Many isochromats' sums have no bias from the sines and cosines, be a sample's
    factor one pair (every 16th sample), two, or no phase at all (in phase, without
    field, decay or gradient).  A pair is 3.2e-8 short on average: the bar is half of
    that, far above what is left of the single roundings (1e-7 / sqrt(K))."""
    K, n_read, g = 200000, 48, 0.02
    rng = np.random.default_rng(17)
    f = lambda v: np.ascontiguousarray(v, np.float32)
    still = case == "no phase"
    ph = synth.Phantom(f(rng.uniform(-0.1, 0.1, K)), f(np.zeros(K)), f(rng.uniform(-1e-3, 1e-3, K)),
                       f(rng.uniform(0.6, 1.0, K)), f(np.full(K, 1e20) if still else rng.uniform(0.05, 0.09, K)),
                       f(np.zeros(K) if still else rng.uniform(-40, 40, K)), f(rng.uniform(0.5, 1.0, K)))
    sb = SeqBuilder(1e-6, "bias")
    sb.rf(synth.sinc_pulse(200, 1e-6, 0.5), (0.0, 0.0, 0.01))
    if still:
        sb.adc(4 * n_read, (0.0, 0.0, 0.0), 4 * np.arange(n_read) + 2)
        at = np.arange(n_read)
    else:
        at = np.array([int(case.split()[1])])
        sb.relax(2e-3, (-g * (4 * at[0] + 2) * 1e-6, 0.0, -1e-6))
        sb.adc(4 * n_read, (g, 0.0, 0.0), 4 * np.arange(n_read) + 2)
    sim = gb.Simulator(0)
    sim.set_phantom(ph)
    sim.set_sequence(sb.build())
    s = sim.simulate(gb.GBS_CACHED)[1].cpu().numpy()[at]
    ref = sim.simulate(gb.GBS_PLAIN)[1].cpu().numpy()[at]
    sim.close()
    bias = ((s - ref) / ref).real
    print(f"[gpu] cached readouts, {case}: bias {bias.min():.2e} .. {bias.max():.2e}, "
          f"|S| {np.abs(ref).min() / ph.m0.sum():.2f}", flush=True)
    assert np.abs(bias).max() <= 1.6e-8
