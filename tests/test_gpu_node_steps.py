"""Node-weight fits cut into launches of any length give the same bits: the draws
pass through blocks of 16 generations that start at multiples of 16, node sets
change at multiples of 16, and the stretches of the generation loop end at
multiples of 8, wherever a launch begins and ends.
"""
import numpy as np
import pytest

import synth
from gpu_util import block_of, ctx, settings_of, to_dev
from paper_1906_10598_amd import phasetrack as ptk
from test_gpu_nodes import _block, _fit, _same

pytestmark = pytest.mark.gpu


def _settings(P, gens, window):
    return ptk.make_settings(pop=P, max_gens=gens, F=0.5, CR=0.9, seed=5, rel_tol=1e-9 if window else 0.0,
                             window=50 if window else 0)


def _served(blk, de, step):
    srv = ptk.pt_server_create(ctx().handle, ptk.make_server_config(de, max_slots=2, gens_per_step=step))
    try:
        ptk.pt_server_submit(srv, 0, blk)
        for _ in range(2000):
            ptk.pt_server_step(srv, ptk.current_stream())
            got = ptk.pt_server_poll(srv)
            if got:
                return got[0].fit
    finally:
        ptk.pt_server_destroy(srv)


@pytest.mark.parametrize("step", [1, 5, 7, 8, 9, 15, 16, 17, 24, 33, 100, 513, 700])
@pytest.mark.parametrize("P,window", [(40, False), (40, True), (9, False), (64, True), (130, False)])
def test_any_cut_into_launches(P, window, step):
    b = synth.config1(1, n=20_000)
    blk = block_of(b, to_dev(b.samples))
    de = _settings(P, 203, window)
    want = ctx().fit_block(blk, de)  # one launch
    assert ptk.pt_ctx_fit_launches(ctx().handle) == 1
    got = _served(blk, de, step)
    assert list(got.coef) == list(want.coef)
    assert (got.objective, got.generations, got.flags) == (want.objective, want.generations, want.flags)


@pytest.mark.parametrize("margin", [1e-2, 1e-4, 1e-6])
def test_abandoned_late(margin):
    """A fit whose best sinks below the signal-to-noise limit only as it converges
    (by then on the smallest node set, its waves at different points) is run again
    over its samples: the noise is tuned so that the final best lies `margin` below
    the limit.
    """
    clean = _block(20_000, sigma=0.0, dtype=np.float64)
    noise = np.random.default_rng(8).standard_normal(clean.n)
    s0 = clean.samples.copy()
    de = settings_of(clean, gens=900)

    def over_samples(sigma):
        clean.samples = s0 + sigma * noise
        pb = block_of(clean, to_dev(clean.samples))
        got = _fit([pb], de, ptk.PT_LAUNCH_GRAPH)
        return pb, got, got[0][0].objective / float(np.sum(clean.samples ** 2)) / 1e-3

    sigma, want = 0.03 * float(np.std(s0)), 1.0 - margin
    for _ in range(6):  # (the ratio goes with the noise's power but for 1e-3 of it)
        _, _, r = over_samples(sigma)
        sigma *= (want / r) ** 0.5
    pb, ref, r = over_samples(sigma)
    assert 0.5 * margin < 1.0 - r < 2.0 * margin
    _same(_fit([pb], de), ref, margin)
