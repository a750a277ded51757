"""The per-run form errs by no more than the sweep over the isochromats that it
takes the place of (a call with (0, 0, M0) given explicitly): final state and
signal against the FP64 oracle, root mean square over scans of different numbers
of lines, a tenth allowed for chance."""
import numpy as np
import pytest

import oracle
from test_gpu_runs import gb, grouped, phantom, sequence  # noqa: F401  (gb: fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,lines,kw", [
    ("up to 128 lines", [24, 57, 100, 112, 128], {}),
    ("more lines", [136, 200, 256, 300], {}),
    ("final y moment", [20, 40, 60, 80], dict(rewind=False, end_ky=7.25)),
])
def test_no_larger_than_the_sweep(gb, name, lines, kw):  # noqa: F811
    sq = np.zeros((2, 2))
    for n in lines:
        ph = phantom(12, 60, 4, seed=n, classes=3)
        seq = sequence(range(-(n // 2), n - n // 2), n_read=6, rf_steps=64, **kw)
        Mr, sr = oracle.simulate(ph, seq)
        for q, explicit in enumerate((False, True)):
            M, s = grouped(gb, ph, seq, explicit=explicit)
            sq[q] += np.linalg.norm(M - Mr) ** 2 / np.linalg.norm(Mr) ** 2, np.linalg.norm(s - sr) ** 2 / np.linalg.norm(sr) ** 2
    runs, sweep = np.sqrt(sq / len(lines))
    print(f"[gpu] errors, {name}: M by runs {runs[0]:.2e}, swept {sweep[0]:.2e}; signal {runs[1]:.2e}, {sweep[1]:.2e}", flush=True)
    assert (runs <= 1.1 * sweep).all()


@pytest.mark.parametrize("lines", [64, 120, 250])
def test_amplitude(gb, lines):  # noqa: F811
    """The phases of a run's lines are products of several hardware sine/cosine
    pairs, each short by 3.2e-8 on average: the amplitude of the signal (its part
    along the oracle's) may be off by what the sweep's is and one FP32 rounding,
    2^-24.  A phantom far larger than a pixel, so that the phases cover the turn."""
    off = np.zeros(2)
    for seed in range(4):
        ph = phantom(10, 160, 2, seed=seed)
        seq = sequence(range(-(lines // 2), lines - lines // 2), n_read=2, rf_steps=32)
        _, sr = oracle.simulate(ph, seq)
        for q, explicit in enumerate((False, True)):
            _, s = grouped(gb, ph, seq, explicit=explicit)
            off[q] += abs(np.vdot(sr, s).real / np.vdot(sr, sr).real - 1.0) / 4
    print(f"[gpu] amplitude, {lines} lines: by runs off by {off[0]:.2e}, swept {off[1]:.2e}", flush=True)
    assert off[0] <= off[1] + 2.0 ** -24
