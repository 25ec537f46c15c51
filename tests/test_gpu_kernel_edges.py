"""Edges of the kernels' tiles, splits and dispatch rules: the sizes at which
a kernel's remainder handling or the choice of its form changes, against the
FP64 oracle (tests/test_gpu_parity.py and its neighbours cover the values at
ordinary sizes)."""

import numpy as np
import pytest

import oracle

from gpu_util import ctx

pytestmark = pytest.mark.gpu


# ------------------------------------------------------------ conditioning

@pytest.mark.parametrize("L", [64, 128, 256, 512, 1024, 2048, 4096])
def test_condition_transform_lengths(L):
    """Every transform length (all remainders of its stage count by three),
    blocks of one sample up to several segments and one sample past them, and
    segment counts around the 128-segment tile of the PSD sum.  Tolerance: an
    FP32 transform pair of 2 log2(L) <= 24 stages, each of 2^-24 relative,
    on values up to ~30: below 24 * 6e-8 * 30 = 4e-5."""
    from paper_2410_16416_amd import lloid
    rng = np.random.default_rng(1000 + L)
    given = 2.0 / 1024 * (1.0 + 0.5 * np.cos(np.linspace(0, np.pi, L // 2 + 1)))
    for n in (1, L // 2, L - 1, L, L + 1, 3 * L + 17, 64 * L, 64 * L + L // 2 + 3):
        x = rng.standard_normal(n) * 2.0
        psd = given if n < L else None
        out, got, gated = lloid.lloid_condition(ctx(), 1024, x, L, psd=psd)
        want_psd = oracle.welch_psd(x, 1024, L) if psd is None else given
        # one segment's bins may nearly vanish: the gain there is large, so the
        # reference whitens with the PSD the device reports
        want = oracle.whiten(x, 1024, L, got)
        assert gated == 0
        assert np.max(np.abs(got - want_psd)) <= 1e-5 * want_psd.max()
        assert np.max(np.abs(out - want)) <= 4e-5 * max(1.0, np.max(np.abs(want)) / 30.0), n


@pytest.mark.parametrize("half", [0, 1, 63, 64, 700, 32600, 33000, 10 ** 6])
def test_gate_reach(half):
    """Half widths around a bitmap word, around the reach that fits a
    workgroup's LDS copy of the bitmap (1024 words) and past the block, with
    loud samples at both ends."""
    from paper_2410_16416_amd import lloid
    L, thr = 256, 20.0
    x = np.random.default_rng(77).standard_normal(150001)
    for n0 in (0, 511, 512, 75000, 150000):
        x[n0] += 4000.0
    flat = np.full(L // 2 + 1, 2.0 / 1024)     # the identity: white noise of unit variance
    out, _, gated = lloid.lloid_condition(ctx(), 1024, x, L, thr, half, psd=flat)
    want, count = oracle.gate(oracle.whiten(x, 1024, L, flat), thr, half)
    assert gated == count
    assert np.array_equal(out == 0, want == 0)
