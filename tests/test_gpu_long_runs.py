"""Runs of many members in the per-run form of the grouped simulation: the sum
of a run's M0 exp(-i phi_y) may not lose precision with the run's length.  M0 is
the same for every member, so that the roundings of a long FP32 sum all go one
way.

Reference: the members of a run differ in y alone, and no y moment precedes a
pulse, so a readout is the FP64 oracle's signal of one member of the run times
the sum of exp(-2 pi i c y) over the run, c the readout's phase encode.

Bar (relative L2 over all samples): 5e-6.  FP32 sums of 32 equal terms err by
up to 32 half-ulps, 1.9e-6 of the sum; the FP32 state of 16 excitations and the
phases' products account for the rest."""
import numpy as np
import pytest

import oracle
import synth
from synth import GAMMA_BAR
from test_gpu_runs import gb, grouped, sequence  # noqa: F401  (gb: fixture)

pytestmark = pytest.mark.gpu

FOV = 0.2  # of sequence()'s phase encodes
TOL = 5e-6


def column_phantom(R, L, x=None):
    """R runs of L members: x differs from run to run, y inside a run."""
    x = np.linspace(-0.02, 0.02, R) if x is None else x
    y = (np.arange(L) + 0.5) / L * FOV - FOV / 2
    f = lambda v: np.ascontiguousarray(v, np.float32)
    one = np.ones(R * L)
    return synth.Phantom(f(np.repeat(x, L)), f(np.tile(y, R)), f(0 * one), f(0.9 * one), f(0.08 * one), f(0 * one),
                         f(0.85 * one))


def reference(ph, R, L, seq, ky):
    """Signal of R runs of L members each under sequence(ky)."""
    first = synth.Phantom(*(np.ascontiguousarray(v[::L]) for v in (ph.x, 0 * ph.y, ph.z, ph.t1, ph.t2, ph.df, ph.m0)))
    _, s = oracle.simulate(first, seq)
    y = ph.y[:L].astype(np.float64)
    w = np.array([np.exp(-2j * np.pi * k / FOV * y).sum() for k in ky])
    return (np.asarray(s).reshape(len(ky), -1) * w[:, None]).reshape(-1)


@pytest.mark.parametrize("R,L", [(3, 31), (3, 32), (3, 33), (5, 96), (40, 1000), (2, 16384), (1, 131072), (9, 40000)])
@pytest.mark.parametrize("name,ky", [("no encode", [0] * 16), ("encoded", [0, 1, 0, -1, 0, 2, 0, 3, 0, 40, 0, -70, 0, 0, 1, 0])])
def test_equal_terms(gb, R, L, name, ky):  # noqa: F811
    ph = column_phantom(R, L)
    seq = sequence(ky)
    print(f"[gpu] long runs R={R} L={L} {name}", flush=True)
    _, s = grouped(gb, ph, seq)
    ref = reference(ph, R, L, seq, ky)
    rel = float(np.linalg.norm(s - ref) / np.linalg.norm(ref))
    print(f"[gpu] long runs R={R} L={L} {name}: rel {rel:.2e}", flush=True)
    assert rel <= TOL, (R, L, name, rel)


@pytest.mark.parametrize("sizes", [[1023], [1024], [1025], [1534, 1], [1, 1534], [2, 1535, 7], [511, 512, 513, 1024],
                                   [5000], [3, 2048, 3, 2047, 9, 700, 4096]])
@pytest.mark.parametrize("axis", [(0, 0, 1), (0.3, 0, 1)])
def test_pieces(gb, sizes, axis):  # noqa: F811
    """Runs around the length from which they are cut: state and signal, with
    transitions per z-group and per run, and the count of two-axis groups."""
    rng = np.random.default_rng(len(sizes))
    x = np.repeat(np.linspace(-0.02, 0.02, len(sizes)), sizes)
    K = x.size
    f = lambda v: np.ascontiguousarray(v, np.float32)
    order = rng.permutation(K)
    ph = synth.Phantom(f(x[order]), f(rng.uniform(-0.1, 0.1, K)), f(0 * x + 1e-3), f(0 * x + 0.9), f(0 * x + 0.08),
                       f(0 * x + 5.0), f(rng.uniform(0.1, 1.0, K)))
    seq = sequence(range(-5, 6), rf_axis=axis)
    Mr, sr = oracle.simulate(ph, seq)
    sim = gb.Simulator(0)
    sim.set_phantom(ph)
    sim.set_sequence(seq)
    sim.build_groups()
    assert sim.info()["n_xz_groups"] == len(sizes)
    sim.close()
    for explicit in (False, True):  # by runs, and the sweep over the isochromats
        M, s = grouped(gb, ph, seq, explicit=explicit)
        dm, rel = float(np.max(np.abs(M - Mr))), float(np.linalg.norm(s - sr) / np.linalg.norm(sr))
        print(f"[gpu] pieces {sizes} {axis} explicit={explicit}: max|dM|={dm:.2e} rel {rel:.2e}", flush=True)
        assert dm <= 1e-5 and rel <= 1e-4, (sizes, axis, explicit, dm, rel)


@pytest.mark.parametrize("R", [1, 8])
def test_long_runs_fill_the_chip(gb, R):  # noqa: F811
    """2^18 isochromats in one or eight runs take no more than four times as long
    as in 256 runs (one wavefront per run: 14 to 60 times as long)."""
    import time
    import torch

    def us(R):
        sim = gb.Simulator(0)
        sim.set_phantom(column_phantom(R, (1 << 18) // R))
        sim.set_sequence(sequence(range(-8, 8)))
        sim.build_groups()
        best = 1e9
        for _ in range(6):
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(5):
                sim.simulate(gb.GBS_GROUPED)
            torch.cuda.synchronize()
            best = min(best, (time.perf_counter() - t) / 5 * 1e6)
        sim.close()
        return best

    few, many = us(R), us(256)
    print(f"[gpu] 2^18 isochromats in {R} runs {few:.1f} us, in 256 {many:.1f} us", flush=True)
    assert few <= 4.0 * many
