"""Fits through node weights (the automatic launch mode) against the launch
forms that evaluate every sample (PT_LAUNCH_GRAPH).

The two differ only in how the objective is summed: by at most the phasor
path's stated per-sample error on one side and a few ulp of the samples'
energy on the other.  Over the first generations no selection compares
objectives that close, so populations are identical and objectives agree
within that tolerance (1e-10 relative, the tolerance of the objective tests).
What node weights do not carry -- samples that are not finite, more than
30 dB of signal to noise, boxes too wide, populations above 240 -- runs the
other forms and equals them bit for bit.
"""
import math

import numpy as np
import pytest

import oracle
import synth
from gpu_util import assert_chi2_close, block_of, ctx, model_phase_err, settings_of, to_dev
from paper_1906_10598_amd import phasetrack as ptk

pytestmark = pytest.mark.gpu


def _fit(pbs, de, mode=ptk.PT_LAUNCH_AUTO, fusion=ptk.PT_FUSION_AUTO, timing=False):
    c = ctx()
    ptk.pt_ctx_set_launch_mode(c.handle, mode)
    ptk.pt_ctx_set_step_fusion(c.handle, fusion)
    ptk.pt_ctx_set_timing(c.handle, timing)
    try:
        fits = c.fit_batch(pbs, de) if len(pbs) > 1 else [c.fit_block(pbs[0], de)]
        out = []
        for k, f in enumerate(fits):
            pop, fpop = ptk.pt_last_population(c.handle, k, de.pop)
            out.append((f, pop, fpop, ptk.pt_last_history(c.handle, k, f.generations + 1)))
    finally:
        ptk.pt_ctx_set_timing(c.handle, False)
        ptk.pt_ctx_set_step_fusion(c.handle, ptk.PT_FUSION_AUTO)
        ptk.pt_ctx_set_launch_mode(c.handle, ptk.PT_LAUNCH_AUTO)
    return out


def _same(a, b, label=""):
    for x, y in zip(a, b):
        assert list(x[0].coef) == list(y[0].coef), label
        assert np.array_equal(x[0].objective, y[0].objective, equal_nan=True), label
        assert x[0].generations == y[0].generations and x[0].flags == y[0].flags, label
        for p, q in zip(x[1:], y[1:]):
            assert np.array_equal(p, q, equal_nan=True), label


def _close(a, b, n, amp, label):
    """Identical populations, objectives within the objective tests' tolerance."""
    floor = model_phase_err()
    (fa, pa, va, ha), (fb, pb, vb, hb) = a, b
    print(f"[nodes {label}] objective rel diff {abs(fa.objective - fb.objective) / fb.objective:.1e}", flush=True)
    assert np.array_equal(pa, pb), label
    assert fa.generations == fb.generations and fa.flags == fb.flags, label
    assert list(fa.coef) == list(fb.coef), label
    assert_chi2_close(va, vb, n, amp=amp, floor=floor)
    assert_chi2_close(ha, hb, n, amp=amp, floor=floor)


def _block(n, fs=50_000.0, x=(0.7, 1.3, 1234.5, 2.5, 0.02, 0.0, 0.0), half=(0.1, 3.0, 0.5, 0.1, 0.01, 0.0, 0.0),
           sigma=0.4, ref=None, dtype=np.float32, seed=0):
    x, half = np.array(x, dtype=float), np.array(half, dtype=float)
    ref = n / 2 if ref is None else ref
    t = (np.arange(n) - ref) / fs
    ph = x[1] + 2 * np.pi * (x[2] * t + x[3] * t ** 2 / 2 + x[4] * t ** 3 / 6 + x[6] * t ** 4 / 24)
    s = (x[0] + x[5] * t) * np.cos(ph) + np.random.default_rng(seed).normal(0, sigma, n)
    return synth.Block(s.astype(dtype), fs, ref, x, x - half, x + half, synth.DESettings(40, 20, seed=7 + seed), sigma,
                       stream=seed, name=f"n{n}")


# tile and workgroup edges, one tile, several runs per workgroup; short and long spans
@pytest.mark.parametrize("n", [64, 65, 100, 4095, 4096, 4097, 8192 + 5, 65536 + 33, 400_001, 4 * 1024 * 1024 + 4097])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_block_lengths(n, dtype):
    b = _block(n, dtype=dtype)
    pb = block_of(b, to_dev(b.samples))
    de = settings_of(b, gens=12)
    _close(_fit([pb], de)[0], _fit([pb], de, ptk.PT_LAUNCH_GRAPH)[0], n, 0.8, f"n {n}")


# one, two and four members per row of lanes, and the first population past them
@pytest.mark.parametrize("pop", [4, 5, 40, 59, 60, 61, 120, 121, 240, 241])
def test_populations(pop):
    b = synth.config0(1)
    pb = block_of(b, to_dev(b.samples))
    de = settings_of(b, gens=15, pop=pop)
    a, g = _fit([pb], de)[0], _fit([pb], de, ptk.PT_LAUNCH_GRAPH)[0]
    if pop > 240:
        _same([a], [g])
    _close(a, g, b.n, 1.2, f"pop {pop}")


FORMS = {
    "slope": dict(x=(0.7, 1.3, 1234.5, 2.5, 0.02, 0.03, 0.0), half=(0.1, 3.0, 0.5, 0.1, 0.01, 0.05, 0.0)),
    "quartic": dict(x=(0.7, 1.3, -8234.5, 2.5, 0.02, 0.0, 5e-4), half=(0.1, 3.0, 0.5, 0.1, 0.01, 0.0, 2e-4)),
    "slope-quartic": dict(x=(0.7, 1.3, 19_000.5, -4.5, 0.02, 0.03, 5e-4), half=(0.1, 3.0, 0.5, 0.1, 0.01, 0.05, 2e-4)),
    "carrier near zero": dict(x=(0.7, 1.3, 5.0, 0.0, 0.0, 0.0, 0.0)),
    "carrier near Nyquist": dict(x=(0.7, 1.3, 24_995.0, 0.0, 0.0, 0.0, 0.0)),
    "fixed rate": dict(half=(0.1, 3.0, 0.5, 0.0, 0.0, 0.0, 0.0)),
    "fixed amplitude": dict(half=(0.0, 3.0, 0.5, 0.1, 0.01, 0.0, 0.0)),
    "wide": dict(half=(0.1, 3.0, 8.0, 0.5, 0.05, 0.0, 0.0)),
    "reference at the start": dict(ref=0.0),
    "reference outside": dict(ref=-150_000.25),
}


@pytest.mark.parametrize("objective", [ptk.PT_OBJ_CHI2, ptk.PT_OBJ_COR])
@pytest.mark.parametrize("form", list(FORMS))
def test_models_and_references(form, objective):
    b = _block(200_003, **FORMS[form])
    pb = block_of(b, to_dev(b.samples))
    de = settings_of(b, gens=15, objective=objective)
    a, g = _fit([pb], de)[0], _fit([pb], de, ptk.PT_LAUNCH_GRAPH)[0]
    if objective == ptk.PT_OBJ_COR:
        # F = 1 / (arctan C + pi / 2) is flat in C here: dF <= dC F^2 / (1 + C^2)
        assert np.array_equal(a[1], g[1])
        assert np.max(np.abs(a[2] - g[2])) < 1e-12 and np.max(np.abs(a[3] - g[3])) < 1e-12
    else:
        _close(a, g, b.n, 1.0, form)


def test_objectives_match_the_oracle_along_the_fit():
    # before and after the population has drawn together (the narrow node set),
    # and across launches of 500 generations
    b = synth.config1(0)
    pb = block_of(b, to_dev(b.samples))
    s64 = b.samples.astype(np.float64)
    for gens in (0, 1, 40, 150, 499, 500, 501, 1100):
        f, pop, fpop, hist = _fit([pb], settings_of(b, gens=gens))[0]
        idx = [0, 17, 39]
        want = oracle.chi2_pop(s64, b.fs, b.ref, pop[idx])
        err = np.max(np.abs(fpop[idx] - want) / want)
        print(f"[nodes {gens} generations] worst objective error {err:.1e}", flush=True)
        # S2 = 2 chi^2 at 0 dB: a few ulp of each of ~100 terms, and the oracle's own phase rounding
        assert err < 1e-12
        assert len(hist) == gens + 1 and hist[-1] == f.objective == fpop.min()
        assert np.all(pop >= b.lo) and np.all(pop <= b.hi)


def test_launch_chunks_do_not_change_a_fit():
    # one generation per launch (timing) against 500, with the window rule and without
    b = synth.config0(3)
    pb = block_of(b, to_dev(b.samples))
    for kw in (dict(gens=130), dict(gens=900, rel_tol=1e-9, window=30), dict(gens=300, rel_tol=1e-3, window=1)):
        de = settings_of(b, **kw)
        a, t = _fit([pb], de), _fit([pb], de, timing=True)
        _same(a, t, str(kw))
        assert (a[0][0].flags & ptk.PT_FLAG_CONVERGED) == (ptk.PT_FLAG_CONVERGED if "window" in kw else 0)


def test_window_longer_than_the_kept_history():
    # a window above 512 generations reads the history from memory
    b = synth.config0(4)
    pb = block_of(b, to_dev(b.samples))
    f, _, _, h = _fit([pb], settings_of(b, gens=3000, rel_tol=1e-6, window=600))[0]
    assert f.flags == ptk.PT_FLAG_CONVERGED
    g = f.generations
    assert h[g - 600] - h[g] <= 1e-6 * h[g]
    assert all(h[k - 600] - h[k] > 1e-6 * h[k] for k in range(600, g))


@pytest.mark.parametrize("case", ["noise-free", "nan", "inf", "too wide"])
def test_what_nodes_do_not_carry_runs_over_the_samples(case):
    b = _block(20_000, sigma=0.0 if case == "noise-free" else 0.4, dtype=np.float64)
    if case in ("nan", "inf"):
        b.samples[777] = math.nan if case == "nan" else math.inf
    if case == "too wide":
        b.lo[2], b.hi[2] = 0.0, 20_000.0
    pb = block_of(b, to_dev(b.samples))
    de = settings_of(b, gens=60)
    _same(_fit([pb], de), _fit([pb], de, ptk.PT_LAUNCH_GRAPH), case)


def test_batch_of_every_kind_equals_its_blocks_alone():
    blocks = [_block(50_000, seed=1), _block(70_001, sigma=0.0, seed=2), synth.config1(2, n=123_457),
              _block(60_000, half=(0.1, 3.0, 400.0, 0.1, 0.01, 0.0, 0.0), seed=3), _block(8000, seed=4,
                                                                                          **FORMS["slope-quartic"])]
    devs = [to_dev(b.samples) for b in blocks]
    pbs = [block_of(b, d) for b, d in zip(blocks, devs)]
    # one geometry, hence one summation order, for the blocks fitted over their samples
    c = ctx()
    ptk.pt_ctx_set_tile(c.handle, 16, 8)
    try:
        for kw in (dict(gens=45), dict(gens=400, rel_tol=1e-7, window=20)):
            de = settings_of(blocks[0], **kw)
            batch = _fit(pbs, de)
            for k, pb in enumerate(pbs):
                _same([batch[k]], _fit([pb], de), str((k, kw)))
    finally:
        ptk.pt_ctx_set_tile(c.handle, 0, 0)


@pytest.mark.parametrize("prec", [ptk.PT_PREC_FP64, ptk.PT_PREC_MIXED])
def test_every_form_over_the_samples_is_bit_identical(prec):
    # step fusion in the explicit graph mode: leading step, last workgroup, automatic, two launches
    blocks = [synth.config1(0, n=60_000), synth.config1(1, n=33_333)]
    devs = [to_dev(b.samples) for b in blocks]
    pbs = [block_of(b, d) for b, d in zip(blocks, devs)]
    for kw in (dict(gens=120), dict(gens=400, rel_tol=1e-9, window=30)):
        de = settings_of(blocks[0], precision=prec, **kw)
        for sel in ([pbs[0]], pbs):
            ref = _fit(sel, de, ptk.PT_LAUNCH_GRAPH, ptk.PT_FUSION_OFF)
            for mode in (ptk.PT_FUSION_LEAD, ptk.PT_FUSION_LAST, ptk.PT_FUSION_AUTO):
                _same(_fit(sel, de, ptk.PT_LAUNCH_GRAPH, mode), ref, str((mode, kw)))
