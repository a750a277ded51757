"""The grouped workspace: gbs_workspace_size is bounded where many groups meet
long readouts, gbs_simulate takes any workspace from the least one on (what the
sweeps and the readouts one by one need) with the same results, and refuses less.
Bars of the other parity tests: |dM| <= 1e-5, relative signal 1e-4."""
import re

import numpy as np
import pytest

import oracle
from test_gpu_readout_products import phantom as many_groups
from test_gpu_readout_products import sequence as readouts
from test_gpu_runs import DM_TOL, SIG_TOL, gb, phantom, sequence  # noqa: F401  (gb: fixture)

pytestmark = pytest.mark.gpu


def least_of(gb, sim):  # noqa: F811
    import torch
    tiny = torch.empty(256, dtype=torch.uint8, device="cuda")
    with pytest.raises(gb.GbsError) as e:
        sim.simulate(gb.GBS_GROUPED, workspace=tiny)
    assert e.value.code == gb.GBS_E_WORKSPACE
    return int(re.search(r"needs (\d+)", str(e.value)).group(1))


def run(sim, gb, n):  # noqa: F811
    import torch
    M, s = sim.simulate(gb.GBS_GROUPED, workspace=torch.empty(n, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    return M.cpu().numpy().astype(np.float64), s.cpu().numpy()


def off(a, b):
    return float(np.max(np.abs(a[0] - b[0]))), float(np.linalg.norm(a[1] - b[1]) / np.linalg.norm(b[1]))


@pytest.mark.parametrize("lines", [3, 40])  # swept in any case; by runs where there is room
def test_least_workspace(gb, lines):  # noqa: F811
    ph, seq = phantom(7, 60, 3), sequence(range(-(lines // 2), lines - lines // 2))
    ref = oracle.simulate(ph, seq)
    sim = gb.Simulator(0)
    sim.set_phantom(ph)
    sim.set_sequence(seq)
    sim.build_groups()
    full, least = sim.workspace_size(gb.GBS_GROUPED), least_of(gb, sim)
    print(f"[gpu] workspace lines={lines}: {full} bytes, least {least}", flush=True)
    assert least <= full and (lines == 3 or least < full)
    for n in sorted({least, (least + full) // 512 * 256, full, full + 4096}):
        dm, rel = off(run(sim, gb, n), ref)
        print(f"[gpu] workspace lines={lines}: {n} bytes: max|dM|={dm:.2e} rel {rel:.2e}", flush=True)
        assert dm <= DM_TOL and rel <= SIG_TOL
    with pytest.raises(gb.GbsError) as e:
        run(sim, gb, least - 1)
    assert e.value.code == gb.GBS_E_WORKSPACE
    sim.close()


@pytest.mark.parametrize("lines,n_read,K", [
    (64, 4096, 200000),  # one tile row takes more than the bound: one by one
    (200, 256, 200000),  # several launches within it
])
def test_bounded_partial_sums(gb, lines, n_read, K):  # noqa: F811
    sim = gb.Simulator(0)
    sim.set_phantom(many_groups(K, 3))
    sim.set_sequence(readouts(lines, n_read))
    sim.build_groups(gb.GBS_AX_X | gb.GBS_AX_Z)
    full, least = sim.workspace_size(gb.GBS_GROUPED), least_of(gb, sim)
    print(f"[gpu] partial sums lines={lines} read={n_read} K={K}: {full} bytes, least {least}", flush=True)
    assert full - least <= (256 << 20) + 4096
    dm, rel = off(run(sim, gb, full), run(sim, gb, least))
    print(f"[gpu] partial sums lines={lines} read={n_read}: between the two max|dM|={dm:.2e} rel {rel:.2e}", flush=True)
    assert dm <= DM_TOL and rel <= SIG_TOL
    sim.close()
