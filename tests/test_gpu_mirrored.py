"""Transitions from half the steps around the length from which the grouped
mode takes them (1024 steps), with B1 along x, along y and between the axes (where
the mirror mixes x and y), and sequences whose pulses take both ways.  One random
state per pulse; bars: the grouped mode rounds the transition's entries to FP32
(four terms, 2.4e-7 of a magnetization up to 1, and the rounding of the output),
6e-7 for each pulse; the cached mode errs by its FP32 output, 2e-7 (for each
pulse's FP32 rows, 2.4e-7 more)."""
import numpy as np
import pytest

import oracle
import synth
from synth import SeqBuilder
from test_gpu_runs import gb  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

PHASE = {"x": 1.0, "y": 1j, "diagonal": (1 + 1j) / np.sqrt(2.0), "other diagonal": (1 - 1j) / np.sqrt(2.0)}


def check(gb, name, pulses, axis=(0.0, 0.0, 1.0)):  # noqa: F811
    import torch
    rng = np.random.default_rng(len(name))
    ph = synth.gre_phantom(15, 5, 4, seed=7)
    ph.m0 = rng.uniform(0.2, 1.0, ph.K).astype(np.float32)
    sb = SeqBuilder(1e-6, name)
    for rf in pulses:
        sb.rf(rf, tuple(0.02 * a for a in axis))
    seq = sb.build()
    m_init = rng.uniform(-0.55, 0.55, (3, ph.K)).astype(np.float32)
    Mr, _ = oracle.simulate(ph, seq, m_init=m_init)
    for mode, bar in ((gb.GBS_GROUPED, 6e-7 * len(pulses)), (gb.GBS_CACHED, 2e-7 + 2.4e-7 * (len(pulses) - 1))):
        sim = gb.Simulator(0)
        sim.set_phantom(ph)
        sim.set_sequence(seq)
        sim.build_groups()
        M, _ = sim.simulate(mode, m_init=torch.from_numpy(m_init))
        torch.cuda.synchronize()
        dm = float(np.max(np.abs(M.cpu().numpy() - Mr)))
        sim.close()
        print(f"[gpu] mirrored {name} mode={mode}: max|dM|={dm:.2e} (bar {bar:.1e})", flush=True)
        assert dm <= bar, (name, mode, dm)


def pulse(n, phase="x", flip=110.0):
    return synth.sinc_pulse(n, 1e-6, np.deg2rad(flip)) * PHASE[phase]


@pytest.mark.parametrize("n", [64, 1023, 1024, 1025, 1087, 2049])
@pytest.mark.parametrize("phase", list(PHASE))
def test_lengths(gb, n, phase):  # noqa: F811
    check(gb, f"{phase} n={n}", [pulse(n, phase)])


@pytest.mark.parametrize("axis", [(0.0, 0.0, 1.0), (1.0, 0.0, 0.0), (0.0, 0.0, 0.0), (0.3, 0.0, 1.0)])
def test_both_ways_in_one_sequence(gb, axis):  # noqa: F811
    bent = pulse(1500, "y", 70.0)
    bent[:9] *= 1.5
    pulses = [pulse(2000, "diagonal", 60.0), pulse(100, "x", 30.0), bent, pulse(1024, "y", 180.0), pulse(1023, "y", 180.0)]
    check(gb, f"mixed {axis}", pulses, axis)
