"""Grouping without a sort (cells of ranked field values) at its limits: fields
with one value, with as many distinct values as the value tables hold (8192)
and one more (then sorted), more cells than the scan takes (then sorted), both
zeros, one isochromat, and K around the workgroup.  Group counts against
numpy's unique over the keys, the simulation against the FP64 oracle (|dM| <=
1e-5, relative signal 1e-4 per readout: the bars of the other parity tests),
which any isochromat in a wrong group or place breaks, as M0 and y are random."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_runs import DM_TOL, SIG_TOL, gb, sequence  # noqa: F401  (gb: fixture)

pytestmark = pytest.mark.gpu


def distinct(n, lo, hi):
    v = np.unique(np.linspace(lo, hi, n).astype(np.float32))
    assert len(v) == n
    return v


def phantom(K, nx=7, nz=5, n1=3, n2=4, nd=3, zeros=False, seed=1):
    """K isochromats over nx x nz positions and n1 x n2 x nd tissue values, every value used."""
    rng = np.random.default_rng(seed)

    def pick(v):
        i = rng.integers(0, len(v), K)
        n = min(len(v), K)
        i[rng.permutation(K)[:n]] = np.arange(n)
        return v[i]

    x, z = pick(distinct(nx, -0.1, 0.1)), pick(distinct(nz, -0.005, 0.005))
    df = pick(distinct(nd, -80.0, 80.0))
    if zeros:  # -0 and +0 are one value
        x, df = np.where(np.abs(x) < 0.04, np.float32(0.0), x), np.where(np.abs(df) < 40, np.float32(0.0), df)
        x[rng.random(K) < 0.5] *= np.float32(-1.0)
        df[(rng.random(K) < 0.5) & (df == 0.0)] *= np.float32(-1.0)
    return synth.Phantom(x, rng.uniform(-0.1, 0.1, K).astype(np.float32), z, pick(distinct(n1, 0.2, 2.0)),
                         pick(distinct(n2, 0.02, 0.3)), df, rng.uniform(0.1, 1.0, K).astype(np.float32))


@pytest.mark.parametrize("name,kw", [
    ("one", dict(K=1, nx=1, nz=1, n1=1, n2=1, nd=1)),
    ("constant", dict(K=700, nx=1, nz=1, n1=1, n2=1, nd=1)),
    ("255", dict(K=255)),
    ("257", dict(K=257)),
    ("zeros", dict(K=3000, zeros=True)),
    ("values-1023", dict(K=20000, nd=1023, n1=2, n2=2)),   # chunk of the rank count less one, and one more
    ("values-1025", dict(K=20000, nd=1025, n1=2, n2=2)),
    ("values-8192", dict(K=20000, nd=8192, n1=1, n2=2)),   # full tables
    ("values-8193", dict(K=20000, nd=8193, n1=1, n2=2)),   # sorted
    ("cells-over", dict(K=20000, nx=4000, nd=40, n1=3, n2=3)),  # 1.4 million cells: sorted
    ("wide-x", dict(K=20000, nx=8192, nz=2, nd=2, n1=2, n2=2)),
])
def test_groups(gb, name, kw):  # noqa: F811
    import torch
    ph, seq = phantom(**kw), sequence(range(-3, 4))
    print(f"[gpu] groups {name}: K={ph.K}", flush=True)
    Mr, sr = oracle.simulate(ph, seq)
    sim = gb.Simulator(0)
    sim.set_phantom(ph)
    sim.set_sequence(seq)
    sim.build_groups(gb.GBS_AX_ALL)
    info = sim.info()
    tissue = [np.asarray(v) + np.float32(0.0) for v in (ph.t1, ph.t2, ph.df)]
    count = lambda *cols: len(np.unique(np.stack(cols + tuple(tissue), 1), axis=0))
    x, y, z = (np.asarray(v) + np.float32(0.0) for v in (ph.x, ph.y, ph.z))
    assert list(info["n_groups"]) == [count(x), count(y), count(z)]
    assert info["n_tissue_groups"] == count() and info["n_xz_groups"] == count(x, z)
    M, s = sim.simulate(gb.GBS_GROUPED)
    torch.cuda.synchronize()
    dm = float(np.max(np.abs(M.cpu().numpy().astype(np.float64) - Mr)))
    n = int(seq.n_samples.max())
    ref, got = np.asarray(sr).reshape(-1, n), s.cpu().numpy().reshape(-1, n)
    rel = np.linalg.norm(got - ref, axis=1) / np.linalg.norm(ref, axis=1)
    print(f"[gpu] groups {name}: max|dM|={dm:.2e} rel per readout {rel.max():.2e}", flush=True)
    assert dm <= DM_TOL and rel.max() <= SIG_TOL
    sim.close()
