"""Edges of the kernels' tiles, splits and dispatch rules: the sizes at which
a kernel's remainder handling or the choice of its form changes, against the
FP64 oracle (tests/test_gpu_parity.py and its neighbours cover the values at
ordinary sizes)."""

import numpy as np
import pytest

import oracle

from workloads import configs
from workloads.bank import SliceSpec

from gpu_util import EPS_ABS, ctx

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


# ------------------------------------------------- decimation, several levels a launch

@pytest.mark.parametrize("level", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("n", [1, 700, 4097, 300000 + 17])
def test_decimated_levels(level, n):
    """A slice at every level (one to three decimation launches: four levels,
    then two at a time), blocks shorter than a workgroup's run and ones of
    many runs, long and short, against the oracle's peaks (FP32 tolerance)."""
    from paper_2410_16416_amd import lloid
    f0 = 4096
    bank = configs.random_basis_bank(8, [SliceSpec(f0, 0, 32, 8), SliceSpec(f0 >> level, 128, 24, 8)], f0,
                                     np.random.default_rng(900 + level))
    x = np.random.default_rng(901 + n).standard_normal(n)
    b = lloid.bank_from_svd(ctx(), bank, "f32")
    try:
        res = lloid.lloid_filter(b, 0, x, window=(1, 4), peaks=True)
    finally:
        lloid.lloid_bank_destroy(b)
    lo = max(0, n - 20000)
    lo -= lo % 1024
    z = oracle.lloid_snr(bank, x, lo, n)
    _, want, _, _ = oracle.peak_table(z, lo, f0, 1, 4)
    assert np.max(np.abs(res.peak_snr[:, lo // 1024:] - want)) < EPS_ABS["f32"]


# ------------------------------------------------- trigger compaction and phases

@pytest.mark.parametrize("templates,windows", [(1, 1), (3, 21), (37, 122), (64, 33), (700, 6100)])
@pytest.mark.parametrize("compute", ["f16", "f32"])
def test_triggers_are_the_peaks_above_threshold(templates, windows, compute):
    """The trigger list against the dense peak tables of the same call, from
    one entry to more compaction blocks (4096) than the offsets are summed
    without a scan for, and few to many entries per wave of the phase kernel:
    the same records in template, window order, the same phases whether every
    entry or only the triggers are asked for."""
    from paper_2410_16416_amd import lloid
    f0, wl = 1024, 8
    bank = configs.random_basis_bank(templates, [SliceSpec(f0, 0, 64, 16)], f0, np.random.default_rng(50))
    for sl in bank.slices:
        sl.mixing *= 2.0 / np.sqrt(np.mean(np.sum(sl.mixing.reshape(templates, -1) ** 2, axis=1)))
    x = np.random.default_rng(51).standard_normal(windows * wl - 3)
    b = lloid.bank_from_svd(ctx(), bank, compute)
    try:
        dense = lloid.lloid_filter(b, 0, x, window=(1, 128), threshold=3.5, peaks=True)
        only = lloid.lloid_filter(b, 0, x, window=(1, 128), threshold=3.5)
    finally:
        lloid.lloid_bank_destroy(b)
    t, w = np.nonzero(dense.peak_snr >= np.float32(3.5))
    for res in (dense, only):
        assert res.n_triggers == t.size
        assert np.array_equal(res.triggers["template_id"], t) and np.array_equal(res.triggers["window"], w)
        assert np.array_equal(res.triggers["snr"], dense.peak_snr[t, w])
        assert np.array_equal(res.triggers["sample"], dense.peak_sample[t, w])
        assert np.array_equal(res.triggers["phase"], dense.peak_phase[t, w])
    assert np.array_equal(dense.triggers, only.triggers)


# ------------------------------------------------- windows shared by workgroups

@pytest.mark.parametrize("compute", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("tail", [0, 1, 255, 256, 257, 1300])
@pytest.mark.parametrize("seconds,win", [(1, (1, 1)), (3, (3, 2)), (2, (1, 16))])
def test_split_windows(compute, tail, seconds, win):
    """Few windows: each is shared by several workgroups, a short last window by
    more than it has column steps.  Peaks against the oracle; the allocation-free
    call and every mixing tile shape (other step widths, other splits) equal bit
    for bit."""
    from paper_2410_16416_amd import lloid
    bank = configs.mini_multirate_bank()
    n = seconds * bank.f0 * 2 + tail
    x = np.random.default_rng(60 + tail).standard_normal(n)
    _, want, at, _ = oracle.peak_table(oracle.lloid_snr(bank, x), 0, bank.f0, *win)
    b = lloid.bank_from_svd(ctx(), bank, compute)
    try:
        res = lloid.lloid_filter(b, 0, x, window=win, peaks=True, threshold=2.5)
        assert np.max(np.abs(res.peak_snr - want)) < EPS_ABS[compute]
        if compute == "f32":
            assert np.mean(res.peak_sample != at) < 0.02   # near ties only
        same = [lloid.lloid_filter_noalloc(b, 0, x, window=win, peaks=True, threshold=2.5)]
        for v in range(1, lloid.MIX_VARIANTS):
            lloid.lloid_ctx_set_tiles(ctx(), 0, v)
            same.append(lloid.lloid_filter(b, 0, x, window=win, peaks=True, threshold=2.5))
    finally:
        lloid.lloid_ctx_set_tiles(ctx(), 0, 0)
        lloid.lloid_bank_destroy(b)
    for r in same:
        assert np.array_equal(r.peak_snr, res.peak_snr) and np.array_equal(r.peak_sample, res.peak_sample)
        assert np.array_equal(r.triggers, res.triggers)


# ------------------------------------------------- narrow FIR tiles

@pytest.mark.parametrize("compute", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("taps", [1, 31, 33, 64, 96, 1023, 1024, 1025, 1088, 2080])
def test_narrow_fir_tiles(compute, taps):
    """Short blocks, whose FIR takes narrow tiles: filters around a chunk (64
    taps), its half and the strain window (1024 taps), basis counts around a
    row tile, columns past a ragged end.  Peaks against the oracle (one filter
    per slice rate), and bit for bit those of every other FIR tile shape, which
    has wide tiles only."""
    from paper_2410_16416_amd import lloid
    f0 = 1024
    l0, l1 = min(taps, 70), min(taps, 130)
    bank = configs.random_basis_bank(70, [SliceSpec(f0, 0, taps, l0), SliceSpec(f0 // 4, 4 * taps, taps, l1)], f0,
                                     np.random.default_rng(70 + taps))
    x = np.random.default_rng(71 + taps).standard_normal(2 * f0 + 129)
    _, want, _, _ = oracle.peak_table(oracle.lloid_snr(bank, x), 0, f0, 1, 2)
    b = lloid.bank_from_svd(ctx(), bank, compute)
    try:
        res = lloid.lloid_filter(b, 0, x, window=(1, 2), peaks=True, threshold=2.5)
        assert np.max(np.abs(res.peak_snr - want)) < EPS_ABS[compute]
        for v in range(1, lloid.FIR_VARIANTS):
            lloid.lloid_ctx_set_tiles(ctx(), v, 0)
            r = lloid.lloid_filter(b, 0, x, window=(1, 2), peaks=True, threshold=2.5)
            assert np.array_equal(r.peak_snr, res.peak_snr) and np.array_equal(r.peak_sample, res.peak_sample)
            assert np.array_equal(r.triggers, res.triggers)
    finally:
        lloid.lloid_ctx_set_tiles(ctx(), 0, 0)
        lloid.lloid_bank_destroy(b)


# ------------------------------------------------- mixing rows held in registers

@pytest.mark.parametrize("compute", ["f16", "bf16"])
@pytest.mark.parametrize("k32", list(range(1, 18)))
def test_register_held_mixing(compute, k32):
    """Every compiled K (32 to 512 and 544), one row tile and
    several, windows of one operand tile, of many and shared between runs, a
    ragged end: peaks against the oracle, and bit for bit those of the
    register-staged tile shapes."""
    from paper_2410_16416_amd import lloid
    f0 = 1024
    bank = configs.random_basis_bank(150 if k32 % 3 else 40, [SliceSpec(f0, 0, 600, 32 * k32 - 16 * (k32 % 2))], f0,
                                     np.random.default_rng(80 + k32))
    x = np.random.default_rng(81).standard_normal(5 * f0 + 77)
    z = oracle.lloid_snr(bank, x)
    b = lloid.bank_from_svd(ctx(), bank, compute)
    try:
        assert lloid.lloid_bank_query(b).concat_k == 32 * k32
        for win in ((1, 1), (1, 32), (1, 10), (4, 3), (6, 1)):
            _, want, _, _ = oracle.peak_table(z, 0, f0, *win)
            lloid.lloid_ctx_set_tiles(ctx(), 0, 0)
            res = lloid.lloid_filter(b, 0, x, window=win, peaks=True, threshold=2.5)
            assert np.max(np.abs(res.peak_snr - want)) < EPS_ABS[compute]
            lloid.lloid_ctx_set_tiles(ctx(), 0, 4)
            r = lloid.lloid_filter(b, 0, x, window=win, peaks=True, threshold=2.5)
            assert np.array_equal(r.peak_snr, res.peak_snr) and np.array_equal(r.peak_sample, res.peak_sample)
            assert np.array_equal(r.triggers, res.triggers)
    finally:
        lloid.lloid_ctx_set_tiles(ctx(), 0, 0)
        lloid.lloid_bank_destroy(b)


@pytest.mark.parametrize("compute", ["f16", "bf16"])
def test_mixing_forms_in_one_call(compute):
    """Banks of several forms of the register-held kernel in one batched call."""
    from paper_2410_16416_amd import lloid
    f0 = 1024
    banks = [configs.random_basis_bank(f, [SliceSpec(f0, 0, 700, l)], f0, np.random.default_rng(90 + l))
             for f, l in ((30, 500), (200, 513), (140, 40), (20, 640), (129, 512))]
    x = np.random.default_rng(91).standard_normal(3 * f0 + 5)
    hs = [lloid.bank_from_svd(ctx(), b, compute) for b in banks]
    try:
        both = lloid.lloid_filter_batch(hs, 0, x, window=(1, 4), peaks=True)
        for k, (h, b) in enumerate(zip(hs, banks)):
            one = lloid.lloid_filter(h, 0, x, window=(1, 4), peaks=True)
            _, want, _, _ = oracle.peak_table(oracle.lloid_snr(b, x), 0, f0, 1, 4)
            assert np.max(np.abs(one.peak_snr - want)) < EPS_ABS[compute]
            assert np.array_equal(both.peak_snr[k], one.peak_snr)
            assert np.array_equal(both.peak_sample[k], one.peak_sample)
    finally:
        for h in hs:
            lloid.lloid_bank_destroy(h)


# ------------------------------------------------- last interpolation hops by group

@pytest.mark.parametrize("compute", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("widths", [(5, 16, 33, 40), (32, 7, 90, 16), (17, 100, 1, 31)])
def test_interpolated_column_blocks(compute, widths):
    """Slices that begin and end inside the operand's 32-column blocks, one or two
    hops of either factor in one launch, blocks that end on either side of a
    column tile, alone and in a batch: peaks against the oracle."""
    from paper_2410_16416_amd import lloid
    f0 = 2048
    specs = [SliceSpec(f0 >> lv, 128 * k, 128, w) for k, (lv, w) in enumerate(zip((0, 1, 2, 3), widths))]
    banks = [configs.random_basis_bank(24, specs[:k], f0, np.random.default_rng(1000 + k)) for k in (4, 2, 3)]
    hs = [lloid.bank_from_svd(ctx(), b, compute) for b in banks]
    try:
        for n in (100, 128, 2048 + 129, 3 * 2048 + 127):
            x = np.random.default_rng(1100 + n).standard_normal(n)
            both = lloid.lloid_filter_batch(hs, 0, x, window=(1, 8), peaks=True)
            for k, (h, b) in enumerate(zip(hs, banks)):
                _, want, _, _ = oracle.peak_table(oracle.lloid_snr(b, x), 0, f0, 1, 8)
                one = lloid.lloid_filter(h, 0, x, window=(1, 8), peaks=True)
                assert np.max(np.abs(one.peak_snr - want)) < EPS_ABS[compute]
                assert np.array_equal(both.peak_snr[k], one.peak_snr)
                assert np.array_equal(both.peak_sample[k], one.peak_sample)
    finally:
        for h in hs:
            lloid.lloid_bank_destroy(h)


# ------------------------------------------------- coincidence over blocks

def _trigger_list(sample, template=0):
    from paper_2410_16416_amd import lloid
    t = np.zeros(len(sample), dtype=lloid.TRIGGER_DTYPE)
    t["sample"], t["template_id"] = sample, template
    t["snr"] = 5.0 + (np.arange(len(sample)) % 7)
    return t


@pytest.mark.parametrize("na,nb", [(0, 0), (0, 257), (1, 0), (255, 1), (256, 256), (257, 255), (513, 4097),
                                   (70000, 70001), (1048576 + 5, 300), (300, 1048576 + 257)])
def test_coincidence_blocks(na, nb):
    """Lists that end on either side of a block, one much longer than the other,
    and more blocks than are added up in place: each trigger of one list pairs
    with the trigger of the other at its time (three times as dense there: the
    neighbours lie outside max_dt); a list out of order anywhere is refused."""
    from paper_2410_16416_amd import lloid
    a, b = _trigger_list(30 * np.arange(na)), _trigger_list(10 * np.arange(nb))
    pairs, bg = lloid.lloid_coincide(ctx(), a, b, 9, background=True)
    n = min(na, -(-nb // 3))
    assert pairs.shape[0] == n
    assert np.array_equal(pairs["a"], np.arange(n)) and np.array_equal(pairs["b"], 3 * np.arange(n))
    want = np.ones(na + nb, dtype=np.uint8)
    want[:n] = 0
    want[na + 3 * np.arange(n)] = 0
    assert np.array_equal(bg, want)
    wide = lloid.lloid_coincide(ctx(), a[:600], b[:600], 25)
    i, j = np.nonzero(np.abs(a["sample"][:600, None] - b["sample"][None, :600]) <= 25)
    assert np.array_equal(wide["a"], i) and np.array_equal(wide["b"], j)
    for lst, k in ((a, na - 1), (b, nb - 1), (a, na // 2), (b, nb // 2)):
        if k > 0:
            keep = lst["sample"][k]
            lst["sample"][k] = lst["sample"][k - 1] - 1
            with pytest.raises(lloid.LloidError):
                lloid.lloid_coincide(ctx(), a, b, 9)
            lst["sample"][k] = keep


@pytest.mark.parametrize("compute", ["f16", "bf16"])
@pytest.mark.parametrize("k", [544, 545, 576, 600, 640, 641, 672])
def test_register_held_mixing_long_k(compute, k):
    """The forms whose last mixing fragments live in the vector registers, with
    k-steps past K (544 and 608), and the first K beyond them: peaks
    against the oracle and bit for bit those of a register-staged tile shape."""
    from paper_2410_16416_amd import lloid
    f0 = 1024
    bank = configs.random_basis_bank(150, [SliceSpec(f0, 0, 700, k)], f0, np.random.default_rng(1200 + k))
    x = np.random.default_rng(1201).standard_normal(4 * f0 + 77)
    z = oracle.lloid_snr(bank, x)
    b = lloid.bank_from_svd(ctx(), bank, compute)
    try:
        for win in ((1, 1), (1, 32), (5, 1)):
            _, want, _, _ = oracle.peak_table(z, 0, f0, *win)
            lloid.lloid_ctx_set_tiles(ctx(), 0, 0)
            res = lloid.lloid_filter(b, 0, x, window=win, peaks=True)
            assert np.max(np.abs(res.peak_snr - want)) < EPS_ABS[compute]
            lloid.lloid_ctx_set_tiles(ctx(), 0, 4)
            r = lloid.lloid_filter(b, 0, x, window=win, peaks=True)
            assert np.array_equal(r.peak_snr, res.peak_snr) and np.array_equal(r.peak_sample, res.peak_sample)
    finally:
        lloid.lloid_ctx_set_tiles(ctx(), 0, 0)
        lloid.lloid_bank_destroy(b)
