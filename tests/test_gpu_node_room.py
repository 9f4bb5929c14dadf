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
