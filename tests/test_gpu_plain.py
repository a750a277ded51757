"""The FP64 stepper at the edges of its step runs and thread layouts: runs of
equal steps (hard pulses, constant gradients) cut by samples, by block ends and
by -0, a run of one step, wide rotations inside a run, and isochromat counts
around a workgroup and around the change from one isochromat per thread to two
(196608).  Against the FP64 oracle; M is rounded to float32 once (|dM| <=
1.2e-7 for |M| <= 1), the signal stays in FP64 (1e-9 of the sum of M0: the
stepper's |B1|^2 is a float32, 6e-8 of it, which enters through the series'
second term, B1 rotations here below 0.02 rad)."""
import numpy as np
import pytest

import oracle
import synth
from synth import SeqBuilder
from test_gpu_runs import gb  # noqa: F401

pytestmark = pytest.mark.gpu


def phantom(K, seed=5):
    rng = np.random.default_rng(seed)
    u = lambda lo, hi: rng.uniform(lo, hi, K).astype(np.float32)
    return synth.Phantom(u(-0.1, 0.1), u(-0.1, 0.1), u(-0.005, 0.005), u(0.2, 2.0), u(0.02, 0.3), u(-80, 80), u(0.1, 1.0))


def sequence(wide):
    """Runs of equal steps; wide: gradients that turn by up to 3 rad per step at |x| = 0.1 m."""
    sb = SeqBuilder(1e-6, "runs")
    g = 3.0 / (2 * np.pi * synth.GAMMA_BAR * 1e-6 * 0.1) if wide else 0.02
    hard = np.full(21, 6e-5 + 2e-5j, np.complex128)
    hard[13] *= 1.5
    sb.rf(hard, (0.01, 0.0, -0.02))
    sb.relax(1e-4, (1e-7, 2e-7, -1e-7))
    sb.adc(40, (g, 0.0, 0.0), [0, 1, 2, 17, 17, 39, 40])
    sb.rf(hard[:13], (0.01, 0.0, -0.02))
    sb.adc(5, (-0.0, 0.01, 0.0), [5])
    sb.adc(5, (0.0, 0.01, 0.0), [0, 3])
    sb.rf(synth.sinc_pulse(30, 1e-6, np.deg2rad(40.0)), (g if wide else 0.0, 0.0, 0.02))
    sb.adc(9, (0.003, 0.0, 0.001), [1, 8])
    return sb.build()


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("K", [1, 63, 255, 256, 257, 513, 196608, 196609])
def test_step_runs(gb, K, wide):  # noqa: F811
    check(gb, f"K={K} wide={wide}", phantom(K), sequence(wide))


@pytest.mark.parametrize("K", [257, 196609])
def test_step_runs_coils(gb, K):  # noqa: F811
    rng = np.random.default_rng(1)
    sens = (rng.uniform(-1, 1, (3, K)) + 1j * rng.uniform(-1, 1, (3, K))).astype(np.complex64)
    check(gb, f"K={K} coils", phantom(K), sequence(True), sens)


def check(gb, name, ph, seq, sens=None):  # noqa: F811
    import torch
    print(f"[gpu] plain {name}", flush=True)
    Mr, sr = oracle.simulate(ph, seq) if sens is None else oracle.simulate_coils(ph, seq, sens)
    sim = gb.Simulator(0)
    sim.set_phantom(ph)
    sim.set_sequence(seq)
    if sens is not None:
        sim.set_coils(sens)
    M, s = sim.simulate(gb.GBS_PLAIN)
    torch.cuda.synchronize()
    dm = float(np.max(np.abs(M.cpu().numpy().astype(np.float64) - Mr)))
    ds = float(np.max(np.abs(s.cpu().numpy() - np.asarray(sr)))) / float(np.sum(ph.m0, dtype=np.float64))
    sim.close()
    print(f"[gpu] plain {name}: max|dM|={dm:.2e} dS={ds:.2e}", flush=True)
    assert dm <= 1.2e-7 and ds <= (1e-9 if sens is None else 2e-9)  # |S(k, p)| <= sqrt(2)
