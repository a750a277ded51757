"""A phantom that is refused after coil sensitivities were set: the next phantom
gets the schedules of one coil (launches of 256 samples), as in a fresh context."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_runs import DM_TOL, SIG_TOL, gb  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def test_refused_phantom_after_coils(gb):  # noqa: F811
    import copy
    import torch
    ph = synth.tiny_phantom(6, 5, 2)
    sb = synth.SeqBuilder(1e-6, "one launch")  # 100 samples during RF: one launch, with 8 coils four
    sb.adc(210, (2e-4, 0.0, 0.0), 2 * np.arange(100) + 1, np.full(210, 2e-5 + 1e-5j))
    seq = sb.build()
    sim = gb.Simulator(0)
    sim.set_phantom(ph)
    sim.set_sequence(seq)
    one = sim.workspace_size(gb.GBS_PLAIN)
    sim.set_coils(synth.coil_maps(ph, 8).astype(np.complex64))
    bad = copy.deepcopy(ph)
    bad.t1[3] = np.nan
    with pytest.raises(gb.GbsError) as e:
        sim.set_phantom(bad)
    assert e.value.code == gb.GBS_E_INVALID
    sim.set_phantom(ph)
    cut = gb.Simulator(0)
    cut.set_phantom(ph)
    cut.set_sequence(seq)
    for mode in (gb.GBS_PLAIN, gb.GBS_CACHED):
        st = [s.simulate(mode, stats=True, flags=gb.GBS_PROFILE)[2] for s in (sim, cut)]
        assert sim.workspace_size(mode) == cut.workspace_size(mode)
        assert all(st[0][k] == st[1][k] for k in ("n_rf_cached", "n_adc_direct", "n_fallback")), st
    assert sim.workspace_size(gb.GBS_PLAIN) == one
    Mr, sr = oracle.simulate(ph, seq)
    for mode in (gb.GBS_PLAIN, gb.GBS_CACHED):
        M, s = sim.simulate(mode)
        torch.cuda.synchronize()
        assert float(np.max(np.abs(M.cpu().numpy() - Mr))) <= DM_TOL
        assert float(np.linalg.norm(s.cpu().numpy() - sr) / np.linalg.norm(sr)) <= SIG_TOL
    sim.close()
    cut.close()
