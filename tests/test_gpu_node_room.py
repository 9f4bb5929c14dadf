"""Fits that find no device memory for their node weights run over their samples
instead, and with little of it in more launches of fewer generations.
"""
import ctypes

import pytest
import torch  # noqa: F401  (its HIP runtime is the one the library is to find)

import synth
from gpu_util import block_of, ctx, settings_of, to_dev
from paper_1906_10598_amd import phasetrack as ptk
from test_gpu_nodes import _fit, _same

pytestmark = pytest.mark.gpu


@pytest.fixture
def room():
    """Sets the bytes one buffer of node weights may take in the tests' context."""
    f = ptk.lib().pt_ctx_node_bytes_
    f.argtypes, f.restype = [ctypes.c_void_p, ctypes.c_uint64], None
    yield lambda n: f(ctx().handle, n)
    f(ctx().handle, 2 ** 64 - 1)


@pytest.mark.parametrize("blocks", [1, 3])
def test_fits_without_room_run_over_their_samples(room, blocks):
    bs = [synth.config1(k, n=30_000 + 1111 * k) for k in range(blocks)]
    devs = [to_dev(b.samples) for b in bs]
    pbs = [block_of(b, d) for b, d in zip(bs, devs)]
    for kw in (dict(gens=150), dict(gens=400, rel_tol=1e-9, window=30)):
        de = settings_of(bs[0], **kw)
        want = _fit(pbs, de, ptk.PT_LAUNCH_GRAPH)
        launches = ptk.pt_ctx_fit_launches(ctx().handle)
        by_nodes = _fit(pbs, de)
        assert ptk.pt_ctx_fit_launches(ctx().handle) == 1
        room(0)
        _same(_fit(pbs, de), want, str(kw))
        assert ptk.pt_ctx_fit_launches(ctx().handle) == launches
        room(2 ** 64 - 1)
        _same(_fit(pbs, de), by_nodes, str(kw))


def test_little_room_takes_more_launches(room):
    b = synth.config0(2)
    pb = block_of(b, to_dev(b.samples))
    de = settings_of(b, gens=1500)
    want = _fit([pb], de)
    assert ptk.pt_ctx_fit_launches(ctx().handle) == 1
    # the draws of 1501 generations of 32 members take 0.4 MB, the weights and the moments
    # of a block of 4096 samples less than 0.25
    room(300_000)
    _same([_fit([pb], de)[0]], want)
    assert ptk.pt_ctx_fit_launches(ctx().handle) > 3


@pytest.mark.parametrize("lead", [False, True])
@pytest.mark.parametrize("room_bytes", [0, 100_000])
def test_served_blocks_without_room_run_over_their_samples(room, lead, room_bytes):
    """No room at all, and room for a block's weights (50 KB with the draws of 2 x 8
    generations) but not for working three blocks' out at once (74 tiles or more of 16
    points and 10 groups of 96 moments, 32 bytes each: 68 KB a block)."""
    bs = [synth.config1(k, n=300_000 + 1111 * k) for k in range(3)]
    devs = [to_dev(b.samples) for b in bs]
    pbs = [block_of(b, d) for b, d in zip(bs, devs)]
    de = settings_of(bs[0], gens=70)
    c = ctx()
    ptk.pt_ctx_set_tile(c.handle, 16, 4)  # the server's geometry
    try:
        want = [_fit([pb], de, ptk.PT_LAUNCH_GRAPH)[0][0] for pb in pbs]
    finally:
        ptk.pt_ctx_set_tile(c.handle, 0, 0)
    ptk.pt_ctx_set_step_fusion(c.handle, ptk.PT_FUSION_LEAD if lead else ptk.PT_FUSION_AUTO)
    srv = ptk.pt_server_create(c.handle, ptk.make_server_config(de, max_slots=4, gens_per_step=8))
    ptk.pt_ctx_set_step_fusion(c.handle, ptk.PT_FUSION_AUTO)
    try:
        room(room_bytes)
        order = {ptk.pt_server_submit(srv, k, pb): k for k, pb in enumerate(pbs)}
        got = {}
        for _ in range(30):
            ptk.pt_server_step(srv, ptk.current_stream())
            for r in ptk.pt_server_poll(srv):
                got[order[r.ticket]] = r.fit
        for k, w in enumerate(want):
            f = got[k]
            assert list(f.coef) == list(w.coef), k
            assert (f.objective, f.generations, f.flags) == (w.objective, w.generations, w.flags), k
    finally:
        ptk.pt_server_destroy(srv)


@pytest.mark.parametrize("mode", [ptk.PT_LAUNCH_AUTO, ptk.PT_LAUNCH_GRAPH])
def test_a_refused_allocation_leaves_no_error_behind(mode):
    """The history of 4096 blocks of 1e7 generations is 328 GB, more than the device has:
    the call says so, and the next one runs."""
    b = synth.config0(5)
    pb = block_of(b, to_dev(b.samples))
    with ptk.Context(0) as c:
        ptk.pt_ctx_set_launch_mode(c.handle, mode)
        with pytest.raises(ptk.PtError, match=r"hipMalloc\(\d+ bytes\) failed"):
            c.fit_batch([pb] * 4096, settings_of(b, gens=10_000_000, pop=4))
        de = settings_of(b, gens=20)
        want = _fit([pb], de, mode)[0][0]
        f = c.fit_block(pb, de)
        assert list(f.coef) == list(want.coef) and f.objective == want.objective
