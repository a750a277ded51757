"""Members at y = 0 in the per-run form: their phases are exact, so the correction
of the sines' and cosines' bias may not touch them.

With y = 0 throughout a phase encode changes nothing, so the lines' signals and
the final state are those of the sequence without it: equal up to half the bias of
one sine/cosine pair (1.6e-8; a line holds up to ten pairs).  Among moving members
the signals are linear in M0: all = still + moving, each computed by itself.  The
FP32 sums of the readout leave random differences of about 1e-7 in a sample; their
mean over 16 lines or more and 4 samples stays within the same bar (a correction
spread over all members by their number shows as 5e-8 and more)."""
import numpy as np
import pytest

import synth
from test_gpu_runs import gb, grouped, sequence  # noqa: F401  (gb: fixture)

pytestmark = pytest.mark.gpu

HALF_PAIR = 1.6e-8


def phantom(R, L, moving):
    """R runs of L members; every third member (none: moving = False) lies off y = 0."""
    rng = np.random.default_rng(R + L)
    f = lambda v: np.ascontiguousarray(v, np.float32)
    K = R * L
    y = np.where((np.arange(K) % 3 == 1) & moving, rng.uniform(-2e-3, 2e-3, K), 0.0)
    one = np.ones(K)
    return synth.Phantom(f(np.repeat(np.linspace(-0.02, 0.02, R), L)), f(y), f(0 * one), f(0.9 * one), f(0.08 * one),
                         f(0 * one), f(rng.uniform(0.5, 1.0, K)))


@pytest.mark.parametrize("lines", [9, 16, 128, 129, 256, 300])
@pytest.mark.parametrize("offset", [0.0, 0.25])
def test_encode_without_extent(gb, lines, offset):  # noqa: F811
    ph = phantom(40, 45, False)
    ky = [offset + k - lines // 2 for k in range(lines)]
    print(f"[gpu] still members, {lines} lines from {ky[0]}", flush=True)
    seq, flat = sequence(ky, end_ky=3.5), sequence([0] * lines, end_ky=3.5)
    flat.moment[-1, 1] = 0.0
    M0, s0 = grouped(gb, ph, flat)
    M1, s1 = grouped(gb, ph, seq)
    bias = ((s1 - s0) / s0).real
    print(f"[gpu] still members, {lines} lines from {ky[0]}: bias {bias.min():.2e} .. {bias.max():.2e}", flush=True)
    assert np.abs(bias).max() <= HALF_PAIR
    assert np.array_equal(M0, M1)


@pytest.mark.parametrize("lines", [16, 128, 256])
def test_still_among_moving(gb, lines):  # noqa: F811
    ph = phantom(900, 45, True)
    seq = sequence([k - lines // 2 for k in range(lines)])
    m0 = ph.m0.copy()
    print(f"[gpu] still among moving, {lines} lines", flush=True)
    s = grouped(gb, ph, seq)[1]
    ph.m0 = np.where(ph.y == 0, m0, np.float32(0))
    still = grouped(gb, ph, seq)[1]
    ph.m0 = np.where(ph.y != 0, m0, np.float32(0))
    part = still + grouped(gb, ph, seq)[1]
    bias = ((s - part) / part).real
    print(f"[gpu] still among moving, {lines} lines: bias {bias.min():.2e} .. {bias.max():.2e}, mean {bias.mean():.2e}", flush=True)
    assert abs(bias.mean()) <= HALF_PAIR
