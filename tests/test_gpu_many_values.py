"""Grouping of phantoms with many distinct field values (a measured dB0 map):
the attempt to group them without a sort is given up on a sample of 12288
isochromats when that holds more than 8192 values.  Group counts against
numpy's unique and the simulation against the FP64 oracle at the sample's edges
(bars of the other parity tests), and the time of a phantom that is given up
against one that the value tables themselves give up."""
import time

import numpy as np
import pytest

import oracle
from test_gpu_groups import phantom
from test_gpu_runs import DM_TOL, SIG_TOL, gb, sequence  # noqa: F401  (gb: fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,nd", [(8192, 8192), (8193, 8193), (12288, 8192), (12288, 8193), (12289, 12289),
                                  (20000, 12288), (20000, 20000), (70000, 70000)])
def test_sampled_fields(gb, K, nd):  # noqa: F811
    import torch
    ph, seq = phantom(K, nd=nd, nx=3, nz=2, n1=1, n2=2), sequence(range(-3, 4))
    print(f"[gpu] many values K={K} nd={nd}", flush=True)
    Mr, sr = oracle.simulate(ph, seq)
    sim = gb.Simulator(0)
    sim.set_phantom(ph)
    sim.set_sequence(seq)
    sim.build_groups(gb.GBS_AX_ALL)
    info = sim.info()
    count = lambda *c: len(np.unique(np.stack(c + (ph.t1, ph.t2, ph.df + np.float32(0.0)), 1), axis=0))
    assert list(info["n_groups"]) == [count(ph.x + np.float32(0.0)), count(ph.y), count(ph.z)]
    assert info["n_tissue_groups"] == count()
    M, s = sim.simulate(gb.GBS_GROUPED)
    torch.cuda.synchronize()
    dm = float(np.max(np.abs(M.cpu().numpy().astype(np.float64) - Mr)))
    rel = float(np.linalg.norm(s.cpu().numpy() - sr) / np.linalg.norm(sr))
    print(f"[gpu] many values K={K} nd={nd}: max|dM|={dm:.2e} rel {rel:.2e}", flush=True)
    assert dm <= DM_TOL and rel <= SIG_TOL
    sim.close()


def test_values_of_their_own_cost_no_more(gb):  # noqa: F811
    """200000 isochromats with a dB0 value each group in at most twice the time of
    the same with 9000 values (both are sorted; the tables filling up under all
    threads took 6 times as long)."""
    import torch
    us = []
    for nd in (200000, 9000):
        sim = gb.Simulator(0)
        sim.set_phantom(phantom(200000, nd=nd, nx=40, nz=3, n1=1, n2=2))
        best = 1e9
        for _ in range(8):
            torch.cuda.synchronize()
            t = time.perf_counter()
            sim.build_groups(gb.GBS_AX_X | gb.GBS_AX_Z)
            torch.cuda.synchronize()
            best = min(best, (time.perf_counter() - t) * 1e6)
        us.append(best)
        sim.close()
    print(f"[gpu] grouping 200000 isochromats: a value each {us[0]:.0f} us, 9000 values {us[1]:.0f} us", flush=True)
    assert us[0] <= 2.0 * us[1]
