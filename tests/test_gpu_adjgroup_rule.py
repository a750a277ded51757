"""The adjoint by groups is taken where the raster steps are worth the grouping
(128 and one per pulse; cells of the fields' values by steps per pulse).  The
edges of its kernels, with a long pulse beside each so that the form is taken,
and the edges of the rule, against the FP64 oracle (bars of the other adjoint
tests: signal and dL/dB1 1e-4, T1 and T2 derivatives 5e-4); and the time of calls
that step either way."""
import time

import numpy as np
import pytest

import oracle
import synth
from test_gpu_adjgroup import CASES, DT, env, phantom, sequence  # noqa: F401  (env: fixture)
from test_gpu_adjoint import make, rel, run, say, tens, wt

pytestmark = pytest.mark.gpu


def check(env, name, ph, t1c, t2c, rf, seq, pb, every):  # noqa: F811
    gb, torch = env
    rng = np.random.default_rng(5)
    w = rng.standard_normal(seq.total_samples) + 1j * rng.standard_normal(seq.total_samples)
    say(f"[gpu] adjoint rule {name}: K={ph.K}, {seq.stepped_count()} stepped steps")
    sim, adj = make(gb, torch, ph, seq, pb, every=every)
    sig, g_rf, g1, g2 = run(adj, torch, rf, t1c, t2c, w)
    sim.close()
    rf32 = rf.real.astype(np.float32) + 1j * rf.imag.astype(np.float32)
    s_o, g_o, g1_o, g2_o = oracle.adjoint(ph, ph.labels, t1c, t2c, seq, rf32, pb, w)
    r = rel(sig, s_o), rel(g_rf, g_o), rel(g1, g1_o), rel(g2, g2_o)
    say(f"[gpu] adjoint rule {name}: signal {r[0]:.2e} dB1 {r[1]:.2e} dT1 {r[2]:.2e} dT2 {r[3]:.2e}")
    assert r[0] <= 1e-4 and r[1] <= 1e-4 and r[2] <= 5e-4 and r[3] <= 5e-4


def pulse(n):
    return synth.sinc_pulse(n, DT, np.deg2rad(60.0)).astype(np.complex128) * np.exp(0.3j)


@pytest.mark.parametrize("every", [256, 8])
@pytest.mark.parametrize("name", CASES)
def test_beside_a_long_pulse(env, name, every):  # noqa: F811
    pk, n_rf, sk = CASES[name]
    ph, t1c, t2c = phantom(**pk)
    rf = np.full(n_rf, 4e-3 * np.exp(0.7j)) if name == "hard" else pulse(n_rf)
    seq, pb = sequence(rf, **{"own": synth.sinc_pulse(400, DT, 0.9), **sk})
    check(env, name, ph, t1c, t2c, rf, seq, pb, every)


@pytest.mark.parametrize("n_rf,lines,pk", [
    (33, 4, dict(K=512)), (32, 4, dict(K=512)),        # 132 and 128 steps of 4 pulses: the first is taken
    (17, 8, dict(K=4096)), (16, 8, dict(K=4096)),      # 136 and 128 of 8
    (16, 9, dict(K=1152)), (16, 9, dict(K=1088)),      # 18 cells, of which 32 and 30 are worth it
    (16, 9, dict(K=648)), (16, 9, dict(K=576)),        # 18 and 16
])
def test_edges(env, n_rf, lines, pk):  # noqa: F811
    ph, t1c, t2c = phantom(**pk)
    rf = pulse(n_rf)
    seq, pb = sequence(rf, lines=lines, n_read=9)
    check(env, f"{lines} x {n_rf} K={ph.K}", ph, t1c, t2c, rf, seq, pb, 64)


def test_short_pulses_cost_no_more(env):  # noqa: F811
    """Three pulses of 16 steps, which could be taken by groups, for 65536
    isochromats in groups of four: no longer than three of 15, which could not, and
    an eighth (by groups a quarter longer)."""
    gb, torch = env
    ph, t1c, t2c = phantom(65536, nz=1365, classes=3, nd=4)
    us = []
    for n_rf in (15, 16):
        seq, pb = sequence(pulse(n_rf), n_read=8)
        sim, adj = make(gb, torch, ph, seq, pb)
        args, w = tens(torch, pulse(n_rf), t1c, t2c), wt(torch, np.ones(seq.total_samples, complex))
        best = 1e9
        for _ in range(10):
            torch.cuda.synchronize()
            t = time.perf_counter()
            adj.forward(*args)
            adj.backward(w)
            torch.cuda.synchronize()
            best = min(best, (time.perf_counter() - t) * 1e6)
        us.append(best)
        sim.close()
    say(f"[gpu] adjoint of 3 short pulses: 15 steps {us[0]:.0f} us, 16 steps {us[1]:.0f} us")
    assert us[1] <= 1.125 * us[0]
