"""The adjoint by groups against the FP64 oracle where it can go wrong: pulses
around the segment length (16 steps), several pulses of which some play the
parameter and some their own B1, samples during RF (pulses between them),
gradients along several axes, wavefronts that hold many groups and groups of
more than a wavefront, samples around the ring of 64, one class and many, and
phantoms on either side of the four isochromats per group from which the form
is taken.  Bars of the other adjoint tests: signal and dL/dB1 1e-4, T1 and T2
derivatives 5e-4 (relative L2)."""
import numpy as np
import pytest

import oracle
import synth
from synth import GAMMA_BAR, SeqBuilder
from test_gpu_adjoint import make, rel, run, say

pytestmark = pytest.mark.gpu

DT = 1e-6


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_03960_amd as gb
    return gb, torch


def phantom(K, nz=3, classes=3, nd=2, nx=0, seed=3):
    """K isochromats: nz (and nx, 0: all different) coordinates, classes and dB0 levels, the rest random."""
    rng = np.random.default_rng(seed)
    lev = lambda n, a: rng.choice(np.linspace(-a, a, n), K)
    u = lambda a: rng.uniform(-a, a, K)
    cls = rng.integers(0, classes, K)
    t1, t2 = np.linspace(0.3, 2.0, classes).astype(np.float32), np.linspace(0.03, 0.3, classes).astype(np.float32)
    f = lambda v: np.asarray(v, np.float32)
    ph = synth.Phantom(f(lev(nx, 0.1) if nx else u(0.1)), f(u(0.1)), f(lev(nz, 0.004)), t1[cls], t2[cls], f(lev(nd, 40.0)),
                       f(rng.uniform(0.2, 1.0, K)), labels=cls.astype(np.int32))
    return ph, t1, t2


def sequence(rf, lines=3, axis=(0, 0, 1), own=None, n_read=20, rf_adc=False):
    """(sequence, parameter blocks): lines of the parameter pulse, own pulses and readouts."""
    sb = SeqBuilder(DT, "groups")
    amp = 0.01
    for i in range(lines):
        sb.rf(rf, tuple(amp * a for a in axis))
        sb.relax(4e-4, tuple(-0.5 * amp * a * len(rf) * DT for a in axis))
        if own is not None:
            sb.rf(own * np.exp(0.5j * (i % 2)), (0.0, 0.0, 0.005))
            sb.relax(1e-4, (1e-8, 0.0, -1e-8))
        n = 4 * n_read + 2
        b1 = np.where(np.arange(n) % 9 < 5, 2e-6 + 1e-6j, 0.0) if rf_adc else None
        sb.adc(n, (2e-4, 0.0, 0.0), 4 * np.arange(n_read) + 1, b1)
        sb.relax(2e-3, (0.0, i / (GAMMA_BAR * 0.2), 1e-7))
    seq = sb.build()
    b = np.nonzero(np.asarray(seq.btype) == synth.BLOCK_RF)[0].astype(np.int32)
    return seq, b if own is None else b[::2]


CASES = {
    "steps-15": (dict(K=700), 15, dict()),
    "steps-16": (dict(K=700), 16, dict()),
    "steps-17": (dict(K=700), 17, dict()),
    "steps-200": (dict(K=1025, nz=1, classes=1, nd=1), 200, dict(lines=2)),
    "own": (dict(K=900), 100, dict(own=synth.sinc_pulse(70, DT, 0.9))),
    "oblique": (dict(K=1500, nx=5), 64, dict(axis=(1, 0, 0.5))),
    "no-gradient": (dict(K=600), 40, dict(axis=(0, 0, 0))),
    "rf-adc": (dict(K=500), 300, dict(rf_adc=True, n_read=6)),
    "rf-adc-short": (dict(K=500), 40, dict(rf_adc=True, n_read=12)),       # too many short pulses: stepped
    "many-classes": (dict(K=4000, classes=64, nd=3), 48, dict(lines=2)),
    "four-per-group": (dict(K=72), 50, dict()),                             # 17 groups
    "under-four": (dict(K=71), 50, dict()),                                 # 18 groups: stepped
    "read-63": (dict(K=400), 33, dict(n_read=63, lines=2)),
    "read-64": (dict(K=400), 33, dict(n_read=64, lines=2)),
    "read-130": (dict(K=400), 33, dict(n_read=130, lines=1)),
    "hard": (dict(K=300), 24, dict()),
}


@pytest.mark.parametrize("every", [256, 8])
@pytest.mark.parametrize("name", CASES)
def test_groups(env, name, every):
    gb, torch = env
    pk, n_rf, sk = CASES[name]
    ph, t1c, t2c = phantom(**pk)
    if name == "hard":  # wide rotations
        rf = np.full(n_rf, 4e-3 * np.exp(0.7j))
    else:
        rf = synth.sinc_pulse(n_rf, DT, np.deg2rad(60.0)).astype(np.complex128) * np.exp(0.3j)
    seq, pb = sequence(rf, **sk)
    rng = np.random.default_rng(5)
    w = rng.standard_normal(seq.total_samples) + 1j * rng.standard_normal(seq.total_samples)
    say(f"[gpu] adjoint groups {name}: K={ph.K}, {seq.stepped_count()} stepped steps")
    sim, adj = make(gb, torch, ph, seq, pb, every=every)
    sig, g_rf, g1, g2 = run(adj, torch, rf, t1c, t2c, w)
    sim.close()
    rf32 = rf.real.astype(np.float32) + 1j * rf.imag.astype(np.float32)
    s_o, g_o, g1_o, g2_o = oracle.adjoint(ph, ph.labels, t1c, t2c, seq, rf32, pb, w)
    r = rel(sig, s_o), rel(g_rf, g_o), rel(g1, g1_o), rel(g2, g2_o)
    say(f"[gpu] adjoint groups {name}: signal {r[0]:.2e} dB1 {r[1]:.2e} dT1 {r[2]:.2e} dT2 {r[3]:.2e}")
    assert r[0] <= 1e-4 and r[1] <= 1e-4 and r[2] <= 5e-4 and r[3] <= 5e-4
