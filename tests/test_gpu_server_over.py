"""The route of served blocks.  Those with more signal to noise than node weights
carry: their fit is run again over the samples, and retries and the track's next
blocks go there at once.  Otherwise the launch mode that a server was created
with decides.
"""
import numpy as np
import pytest

from gpu_util import block_of, ctx, settings_of, to_dev
from paper_1906_10598_amd import phasetrack as ptk
from test_gpu_nodes import _block, _fit

pytestmark = pytest.mark.gpu


def _key(f):
    return list(f.coef) + [f.objective, f.generations, f.flags]


def _serve(srv, track, pb, limit=20):
    """The block's result and the steps it took."""
    ptk.pt_server_submit(srv, track, pb)
    for k in range(limit):
        ptk.pt_server_step(srv, ptk.current_stream())
        got = ptk.pt_server_poll(srv)
        if got:
            return got[0], k + 1
    raise AssertionError("no result")


def _server(de, lead, **kw):
    c = ctx()
    ptk.pt_ctx_set_step_fusion(c.handle, ptk.PT_FUSION_LEAD if lead else ptk.PT_FUSION_AUTO)
    try:
        # one step per fit (the leading step's last launch included); given boxes, no warm start
        return ptk.pt_server_create(c.handle, ptk.make_server_config(de, max_slots=4, gens_per_step=de.max_gens + 2,
                                                                     warm_narrow=0.0, **kw))
    finally:
        ptk.pt_ctx_set_step_fusion(c.handle, ptk.PT_FUSION_AUTO)


@pytest.mark.parametrize("lead", [False, True])
def test_a_track_past_the_limit_and_back(lead):
    sigma = {"high": 0.7 / np.sqrt(2.0) * 10 ** (-50 / 20), "low": 0.3}
    kinds = ["low", "high", "high", "low", "low"]
    bs = [_block(20_000, sigma=sigma[k], dtype=np.float64, seed=q) for q, k in enumerate(kinds)]
    pbs = [block_of(b, to_dev(b.samples)) for b in bs]
    de = settings_of(bs[0], gens=150)
    c = ctx()
    ptk.pt_ctx_set_tile(c.handle, 16, 4)  # the server's geometry
    try:
        over = [_key(_fit([pb], de, ptk.PT_LAUNCH_GRAPH)[0][0]) for pb in pbs]
        auto = [_key(_fit([pb], de)[0][0]) for pb in pbs]
    finally:
        ptk.pt_ctx_set_tile(c.handle, 0, 0)
    assert [a == o for a, o in zip(auto, over)] == [k == "high" for k in kinds]
    srv = _server(de, lead)
    try:
        got, steps = zip(*[_serve(srv, 7, pb) for pb in pbs])
    finally:
        ptk.pt_server_destroy(srv)
    got = [_key(r.fit) for r in got]
    # the second is tried through nodes first; the fourth follows a block past the limit
    assert got == [auto[0], over[1], over[2], over[3], auto[4]]
    assert steps == (1, 2, 1, 1, 1)


@pytest.mark.parametrize("lead", [False, True])
def test_retries_of_a_block_past_the_limit(lead):
    # the amplitude's box misses the truth by half a per cent: the best lies on its bound,
    # past the limit all the same, and the enlarged box holds it
    b = _block(20_000, sigma=1e-3, dtype=np.float64)
    b.lo[0], b.hi[0] = 1.005 * b.truth[0], 1.2 * b.truth[0]
    pb = block_of(b, to_dev(b.samples))
    de = settings_of(b, gens=150)
    srv = _server(de, lead, max_attempts=3, enlarge=2.0)
    try:
        r, steps = _serve(srv, 1, pb)
    finally:
        ptk.pt_server_destroy(srv)
    assert r.attempts == 2 and abs(r.fit.coef[0] - b.truth[0]) < 1e-3
    # tried through nodes once, then over the samples in the first box and the second
    assert steps == 3


@pytest.mark.parametrize("created,later", [(ptk.PT_LAUNCH_AUTO, ptk.PT_LAUNCH_GRAPH),
                                           (ptk.PT_LAUNCH_GRAPH, ptk.PT_LAUNCH_AUTO)])
def test_the_launch_mode_at_creation_holds(created, later):
    b = _block(20_000, dtype=np.float64)
    pb = block_of(b, to_dev(b.samples))
    de = settings_of(b, gens=150)
    c = ctx()
    ptk.pt_ctx_set_tile(c.handle, 16, 4)  # the server's geometry
    try:
        want = {m: _key(_fit([pb], de, m)[0][0]) for m in (created, later)}
    finally:
        ptk.pt_ctx_set_tile(c.handle, 0, 0)
    assert want[created] != want[later]
    ptk.pt_ctx_set_launch_mode(c.handle, created)
    srv = _server(de, False)
    try:
        ptk.pt_ctx_set_launch_mode(c.handle, later)
        assert _key(_serve(srv, 0, pb)[0].fit) == want[created]
    finally:
        ptk.pt_ctx_set_launch_mode(c.handle, ptk.PT_LAUNCH_AUTO)
        ptk.pt_server_destroy(srv)
