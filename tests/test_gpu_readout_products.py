"""Grouped readouts of equal timing as matrix products, at sizes from which they
are taken (1.5e8 terms): full tiles of 64 readouts and parts of one around the
least that is worth a tile (the others are evaluated one by one), samples around
the tile of 128, groups that are no multiple of the stages.  Per readout against
the FP64 oracle, |dM| <= 1e-5 and relative signal 1e-4 (bars of the other parity
tests)."""
import numpy as np
import pytest

import oracle
import synth
from synth import SeqBuilder
from test_gpu_runs import DM_TOL, SIG_TOL, gb  # noqa: F401  (gb: fixture)

pytestmark = pytest.mark.gpu


def phantom(K, seed):
    rng = np.random.default_rng(seed)
    f = lambda v: np.ascontiguousarray(v, np.float32)
    cls = rng.integers(0, 2, K)
    return synth.Phantom(f(np.sort(rng.uniform(-0.1, 0.1, K))), f(rng.uniform(-0.1, 0.1, K)), f(np.full(K, 1e-3)),
                         f(np.array([0.8, 1.3])[cls]), f(np.array([0.05, 0.09])[cls]), f(np.full(K, 4.0)),
                         f(rng.uniform(0.2, 1.0, K)))


def sequence(lines, n_read, odd=0):
    """lines readouts of one timing and odd of another between them."""
    sb = SeqBuilder(1e-6, "products")
    b1 = synth.sinc_pulse(16, 1e-6, np.deg2rad(25.0))
    for i in range(lines + odd):
        sb.rf(b1 * np.exp(0.4j * (i % 5)), (0.0, 0.0, 0.02))
        sb.relax(5e-4, (-2e-8, 0.0, -1.6e-7))
        d = 1 if i % 7 != 3 or i >= 7 * odd else 2
        sb.adc(d * n_read, (5e-3, 0.0, 0.0), d * np.arange(n_read) + 1)
        sb.relax(1e-3, (1e-8, 0.0, 3e-7))
    return sb.build()


@pytest.mark.parametrize("lines,n_read,K,odd", [
    (64, 128, 18500, 0), (64, 127, 18700, 3), (64, 129, 18400, 0), (65, 128, 18433, 0), (111, 128, 18500, 0),
    (112, 128, 18500, 0), (48, 160, 20003, 1), (47, 160, 20003, 0), (56, 64, 42017, 0), (55, 64, 42017, 0),
    (128, 65, 18439, 2), (120, 33, 71000, 0), (192, 32, 24500, 0),
])
def test_products(gb, lines, n_read, K, odd):  # noqa: F811
    import torch
    ph, seq = phantom(K, lines), sequence(lines, n_read, odd)
    print(f"[gpu] readout products lines={lines} read={n_read} K={K}", flush=True)
    Mr, sr = oracle.simulate(ph, seq)
    sim = gb.Simulator(0)
    sim.set_phantom(ph)
    sim.set_sequence(seq)
    sim.build_groups(gb.GBS_AX_X | gb.GBS_AX_Z)
    M, s = sim.simulate(gb.GBS_GROUPED)
    torch.cuda.synchronize()
    dm = float(np.max(np.abs(M.cpu().numpy() - Mr)))
    a, b = s.cpu().numpy().reshape(-1, n_read), np.asarray(sr).reshape(-1, n_read)
    rel = np.linalg.norm(a - b, axis=1) / np.linalg.norm(b, axis=1)
    sim.close()
    print(f"[gpu] readout products lines={lines} read={n_read} K={K}: max|dM|={dm:.2e} rel {rel.max():.2e}", flush=True)
    assert dm <= DM_TOL and rel.max() <= SIG_TOL


def test_few_readouts_of_many_groups(gb):  # noqa: F811
    """Eight readouts of one timing are evaluated like eight of different timings,
    which no product can take: the same time, to a quarter of it (as a product of
    8 of its 64 rows they took 2.5 times as long)."""
    import torch
    ph = phantom(200000, 1)
    ms = []
    for shift in (0, 1):
        sb = SeqBuilder(1e-6, "few")
        for i in range(8):
            sb.rf(synth.sinc_pulse(16, 1e-6, np.deg2rad(25.0)), (0.0, 0.0, 0.02))
            sb.relax(5e-4, (-2e-8, 0.0, -1.6e-7))
            sb.adc(136, (5e-3, 0.0, 0.0), np.arange(128) + shift * i)
            sb.relax(1e-3, (1e-8, 0.0, 3e-7))
        sim = gb.Simulator(0)
        sim.set_phantom(ph)
        sim.set_sequence(sb.build())
        sim.build_groups(gb.GBS_AX_X | gb.GBS_AX_Z)
        ms.append(min(sim.simulate(gb.GBS_GROUPED, stats=True)[2]["ms_adc_eval"] for _ in range(8)))
        torch.cuda.synchronize()
        sim.close()
    print(f"[gpu] 8 readouts of 200000 groups: one timing {ms[0] * 1e3:.0f} us, eight {ms[1] * 1e3:.0f} us", flush=True)
    assert ms[0] <= 1.25 * ms[1]


def test_equal_terms_of_many_groups(gb):  # noqa: F811
    """64 readouts of 100000 groups whose terms are all but equal, so that the
    roundings of a long FP32 sum go one way: as a product (one timing) they err by
    no more than one and a half times what the evaluation one by one errs by
    (readouts shifted by a sample each, which no product takes).

    Reference: no x moment reaches a pulse, so an isochromat differs from the
    oracle's one at x = 0 by exp(-2 pi i m x) at each sample, m its moment there."""
    K, lines, n_read, g = 100000, 64, 128, 1e-7
    x = np.linspace(-0.05, 0.05, K).astype(np.float32)
    one = np.ones(K, np.float32)
    ph = synth.Phantom(x, 0 * x, 0 * x + np.float32(1e-3), 0.8 * one, 0.08 * one, 0 * one, 0.85 * one)
    err = []
    for shift in (0, 1):
        sb = SeqBuilder(1e-6, "equal terms")
        idx = []
        for i in range(lines):
            sb.rf(synth.sinc_pulse(16, 1e-6, np.deg2rad(25.0)), (0.0, 0.0, 0.02))
            sb.relax(5e-4, (0.0, 0.0, -1.6e-7))
            steps = n_read + lines
            idx.append(np.arange(n_read) + shift * i)
            sb.adc(steps, (g, 0.0, 0.0), idx[-1])
            sb.relax(1e-3, (-g * steps * 1e-6, 0.0, 3e-7))
        seq = sb.build()
        first = synth.Phantom(*(np.ascontiguousarray(v[:1]) for v in (0 * x, ph.y, ph.z, ph.t1, ph.t2, ph.df, ph.m0)))
        _, s1 = oracle.simulate(first, seq)
        m = synth.GAMMA_BAR * np.float32(g) * 1e-6 * np.concatenate(idx)
        weight = {v: np.exp(-2j * np.pi * v * x.astype(np.float64)).sum() for v in np.unique(m)}
        ref = np.asarray(s1) * np.array([weight[v] for v in m])
        sim = gb.Simulator(0)
        sim.set_phantom(ph)
        sim.set_sequence(seq)
        sim.build_groups(gb.GBS_AX_X | gb.GBS_AX_Z)
        s = sim.simulate(gb.GBS_GROUPED)[1].cpu().numpy()
        sim.close()
        err.append(float(np.linalg.norm(s - ref) / np.linalg.norm(ref)))
    print(f"[gpu] equal terms of 100000 groups: product {err[0]:.2e}, one by one {err[1]:.2e}", flush=True)
    assert err[0] <= 1.5 * err[1]
