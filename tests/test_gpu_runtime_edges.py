"""Edges of the runtime around the kernels: short trigger windows in streaming
ticks and in chunks, forms of a kernel side by side in one call, the order of
a call's reads on the caller's stream, what a captured tick depends on."""

import numpy as np
import pytest

import oracle

from workloads import configs
from workloads.bank import SliceSpec

from gpu_util import EPS_ABS, ctx
from test_gpu_stream import canon, offline, run_stream

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("compute", ["f16", "bf16"])
@pytest.mark.parametrize("k", [64, 512, 576])
@pytest.mark.parametrize("samples", [32, 64])
def test_short_windows_end_with_the_operand(compute, k, samples):
    """Windows of one or two operand tiles (rings of four and of three tiles),
    where the register-held mixing kernel's loads run ahead over several
    windows: ticks of few windows, and chunks of a few windows each, whose
    operands end with the last one, give the triggers of the whole block bit
    for bit, and those of a tile shape without that kernel."""
    from paper_2410_16416_amd import lloid
    f0, win = 1024, (samples, 1024)
    bank = configs.random_basis_bank(16, [SliceSpec(f0, 0, 600, k)], f0, np.random.default_rng(2000 + k))
    x = np.random.default_rng(2001 + samples).standard_normal(4 * f0 + 5)
    h = lloid.bank_from_svd(ctx(), bank, compute)
    try:
        whole = lloid.lloid_filter(h, 0, x, window=win, threshold=2.0, peaks=True)
        assert whole.n_triggers > 0
        lloid.lloid_ctx_set_chunk_bytes(ctx(), 3 * samples * k * 2)
        parts = lloid.lloid_filter(h, 0, x, window=win, threshold=2.0, peaks=True)
        lloid.lloid_ctx_set_chunk_bytes(ctx(), 6 << 30)
        lloid.lloid_ctx_set_tiles(ctx(), 0, 4)
        other = lloid.lloid_filter(h, 0, x, window=win, threshold=2.0, peaks=True)
        lloid.lloid_ctx_set_tiles(ctx(), 0, 0)
        for r in (parts, other):
            assert np.array_equal(r.triggers, whole.triggers)
            assert np.array_equal(r.peak_snr, whole.peak_snr) and np.array_equal(r.peak_sample, whole.peak_sample)
        s = lloid.lloid_stream_create(ctx(), f0, compute, n_detectors=1, min_rate_hz=f0, window=win, threshold=2.0,
                                      max_filter_s=1.0, max_windows_per_tick=8)
        try:
            slot, active = lloid.lloid_stream_admit(s, h)
            assert active
            got = canon(run_stream(lloid, s, [x], [8 * samples, samples, 5 * samples]))
        finally:
            lloid.lloid_stream_destroy(s)
        assert np.array_equal(got, offline(lloid, h, [x], win, slot, threshold=2.0))
    finally:
        lloid.lloid_ctx_set_chunk_bytes(ctx(), 6 << 30)
        lloid.lloid_ctx_set_tiles(ctx(), 0, 0)
        lloid.lloid_bank_destroy(h)


@pytest.mark.parametrize("seconds", [4, 60])
@pytest.mark.parametrize("strain", ["f64", "f32"])
def test_strain_is_read_in_stream_order(seconds, strain):
    """A context on the caller's stream: a pinned block that an asynchronous copy
    on that stream is still to fill, after some ten milliseconds of other work,
    is filtered as the copy leaves it, small (read where it lies) or large
    (uploaded); the allocation-free call does the same."""
    import torch
    from paper_2410_16416_amd import lloid
    bank = configs.mini_multirate_bank()
    n = seconds * bank.f0 + 3
    dt = torch.float64 if strain == "f64" else torch.float32
    x = torch.randn(n, dtype=dt, generator=torch.Generator().manual_seed(seconds))
    st = torch.cuda.Stream()
    c = lloid.lloid_ctx_create(0, st.cuda_stream)
    try:
        h = lloid.bank_from_svd(c, bank, "f16")
        want = lloid.lloid_filter(h, 0, x.numpy(), window=(1, 4), threshold=2.5, peaks=True)
        assert want.n_triggers > 0
        dev, pinned = x.to("cuda"), torch.empty(n, dtype=dt, pin_memory=True)
        a = torch.randn(4096, 4096, device="cuda")
        torch.cuda.synchronize()
        for call in (lloid.lloid_filter, lloid.lloid_filter_noalloc):
            pinned.zero_()
            with torch.cuda.stream(st):
                for _ in range(20):
                    a = a @ a * 1e-2
                pinned.copy_(dev, non_blocking=True)
            got = call(h, 0, pinned.numpy(), window=(1, 4), threshold=2.5, peaks=True)
            assert np.array_equal(got.triggers, want.triggers) and np.array_equal(got.peak_snr, want.peak_snr)
        lloid.lloid_bank_destroy(h)
    finally:
        lloid.lloid_ctx_destroy(c)


def test_captured_ticks_follow_the_banks_with_lags():
    """Two banks leave a stream with captured ticks and two of the same sizes
    enter, but now it is the one of K = 512 and not the one of K = 256 that
    computes the signal-consistency value: the ticks' buffers and launch sizes
    are the same, the kernel form is not.  Every trigger equals the offline
    one, xi2 included."""
    from paper_2410_16416_amd import lloid
    from workloads import bank_autocorrelation
    f0, win, n = 1024, (1, 4), 12 * 1024
    hs = []
    try:
        for lags in (256, 512):
            for k in (256, 512):
                bank = configs.random_basis_bank(16, [SliceSpec(f0, 0, 600, k)], f0, np.random.default_rng(2100 + k))
                if k == lags:
                    bank.autocorr = bank_autocorrelation(bank, 1)   # one lag: the operands' margins stay as without
                hs.append(lloid.bank_from_svd(ctx(), bank, "f16"))
        x = np.random.default_rng(2101).standard_normal(n)
        s = lloid.lloid_stream_create(ctx(), f0, "f16", n_detectors=1, min_rate_hz=f0, window=win, threshold=2.5,
                                      max_filter_s=1.0, use_graph=True)
        try:
            slots, ends, got = [], [], []
            for pair, (a, b) in enumerate(((0, n // 2), (n // 2, n))):
                for h in hs[2 * pair:2 * pair + 2]:
                    slot, active = lloid.lloid_stream_admit(s, h)
                    assert active
                    slots.append(slot)
                for pos in range(a, b, 256):
                    lloid.lloid_stream_push(s, 0, pos, x[pos:pos + 256])
                    got.append(lloid.lloid_stream_poll(s, wait_ms=-1))
                if pair == 0:
                    ends.append(lloid.lloid_stream_stats_get(s).next_window)
                    for slot in slots:
                        lloid.lloid_stream_remove(s, slot)
            lloid.lloid_stream_flush(s)
            got.append(lloid.lloid_stream_poll(s))
            assert lloid.lloid_stream_stats_get(s).graph_replays > 0
        finally:
            lloid.lloid_stream_destroy(s)
        got = np.concatenate(got)
        for i, (slot, h) in enumerate(zip(slots, hs)):
            w_from, w_to = (0, ends[0]) if i < 2 else (ends[0], None)
            want = offline(lloid, h, [x], win, slot, w_from, w_to, threshold=2.5)
            assert len(want) > 0
            assert np.array_equal(canon(got[got["bank"] == slot]), want), slot
    finally:
        for h in hs:
            lloid.lloid_bank_destroy(h)


@pytest.mark.parametrize("half", [0, 63, 4095, 4096, 262143, 262145, 2 ** 31 - 1])
@pytest.mark.parametrize("loud", [(), (300000,), (0, 599999), tuple(range(5, 600000, 90001))])
def test_gate_reach_over_the_summary_levels(half, loud):
    """Half widths around a word of the loud samples' bits and of each level of
    summary bits (64, 4096 and 262144 samples) and past the block: the gated
    samples and their number are the oracle's; a call without gating is the
    same where nothing is gated."""
    from paper_2410_16416_amd import lloid
    L, thr, n = 256, 20.0, 600000
    x = np.random.default_rng(2200).standard_normal(n)
    x[list(loud)] += 4000.0
    flat = np.full(L // 2 + 1, 2.0 / 1024)     # the identity: white noise of unit variance
    plain, _, _ = lloid.lloid_condition(ctx(), 1024, x, L, psd=flat)
    out, _, gated = lloid.lloid_condition(ctx(), 1024, x, L, thr, half, psd=flat)
    near = np.zeros(n, dtype=bool)
    for k in np.nonzero(np.abs(plain) > thr)[0]:
        near[max(0, k - half):k + half + 1] = True
    assert gated == near.sum() and np.array_equal(out, np.where(near, 0, plain))
    if half < 10 ** 6:
        want, count = oracle.gate(oracle.whiten(x, 1024, L, flat), thr, half)
        assert gated == count and np.array_equal(out == 0, want == 0)


@pytest.mark.parametrize("compute", ["f16", "bf16"])
@pytest.mark.parametrize("samples", [512, 128, 2048])
def test_both_mixing_forms_in_one_call(compute, samples):
    """Banks on both sides of K = 640 in one batched call and in one streaming
    tick: the direct-to-LDS form and the register-held one are two launches over
    one table, with row tiles, splits and item numbers of their own.  The block
    is 32 windows of 512 samples (the split rules then share windows in the
    first form only), 128 of 128 (in neither; in the ticks in the second only) or
    8 of 2048 (in both).  Peaks
    against the oracle, and bit for bit those of the banks alone, of a tile
    shape that takes every bank, and of the ticks."""
    from paper_2410_16416_amd import lloid
    f0, n, win = 1024, 16384, (samples, 1024)
    banks = [configs.random_basis_bank(f, [SliceSpec(f0, 0, 720, k)], f0, np.random.default_rng(2300 + k))
             for f, k in ((129, 500), (100, 672), (200, 40), (90, 700), (300, 640))]
    x = np.random.default_rng(2301).standard_normal(n)
    hs = [lloid.bank_from_svd(ctx(), b, compute) for b in banks]
    try:
        wide = [lloid.lloid_bank_query(h).concat_k > 640 for h in hs]
        assert wide == [False, True, False, True, False]
        both = lloid.lloid_filter_batch(hs, 0, x, window=win, threshold=3.0, peaks=True)
        lloid.lloid_ctx_set_tiles(ctx(), 0, 4)
        other = lloid.lloid_filter_batch(hs, 0, x, window=win, threshold=3.0, peaks=True)
        lloid.lloid_ctx_set_tiles(ctx(), 0, 0)
        assert np.array_equal(both.triggers, other.triggers) and both.n_triggers > 0
        for k, (h, b) in enumerate(zip(hs, banks)):
            one = lloid.lloid_filter(h, 0, x, window=win, threshold=3.0, peaks=True)
            _, want, _, _ = oracle.peak_table(oracle.lloid_snr(b, x[:4096]), 0, f0, *win)
            # (the oracle's block ends at 4096 samples: windows that end before it)
            m = 4096 // samples
            assert np.max(np.abs(one.peak_snr[:, :m] - want[:, :m])) < EPS_ABS[compute]
            for r in (both, other):
                assert np.array_equal(r.peak_snr[k], one.peak_snr)
                assert np.array_equal(r.peak_sample[k], one.peak_sample)
        s = lloid.lloid_stream_create(ctx(), f0, compute, n_detectors=1, min_rate_hz=f0, window=win, threshold=3.0,
                                      max_filter_s=1.0, max_windows_per_tick=4)
        try:
            for h in hs:
                assert lloid.lloid_stream_admit(s, h)[1]
            got = run_stream(lloid, s, [x], [2 * samples])
        finally:
            lloid.lloid_stream_destroy(s)
        assert np.array_equal(canon(got), canon(both.triggers))
    finally:
        lloid.lloid_ctx_set_tiles(ctx(), 0, 0)
        for h in hs:
            lloid.lloid_bank_destroy(h)
