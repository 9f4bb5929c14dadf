"""Samples that go to the device when a block is submitted: the results are those
of blocks that wait in host memory, also where the budget makes them go back.
"""
import numpy as np
import pytest
import torch

from gpu_util import ctx
from paper_1906_10598_amd import phasetrack as ptk
from test_gpu_server import _blk, _key, _settings, _slot_bytes, _stream

pytestmark = pytest.mark.gpu


def _items():
    """Blocks of 100 000, 100 000 (track 0) and 200 000 samples (track 1), in this order."""
    items = _stream(ntracks=3, nblocks=8, seed=6)
    small = [i for i in items if i["block"].n == 100_000]
    large = [i for i in items if i["block"].n == 200_000]
    return [(0, small[0]), (0, small[1]), (1, large[0])]


def _run(blocks, budget, slots=8):
    srv = ptk.pt_server_create(ctx().handle, ptk.make_server_config(_settings(), max_slots=slots, gens_per_step=32,
                                                                    hbm_budget_bytes=budget))
    try:
        order, out, most = {}, {}, 0
        for k, (track, blk) in enumerate(blocks):
            order[ptk.pt_server_submit(srv, track, blk)] = k
        for _ in range(10000):
            a, p = ptk.pt_server_step(srv, ptk.current_stream())
            used = ptk.pt_server_stats(srv)[2]
            assert used <= budget
            most = max(most, a)
            for r in ptk.pt_server_poll(srv):
                out[order[r.ticket]] = _key(r)
            if a == 0 and p == 0:
                break
        return [out[k] for k in range(len(blocks))], most
    finally:
        ptk.pt_server_destroy(srv)


def test_budget_and_origin_of_the_samples():
    items = _items()
    host = [(t, _blk(i)) for t, i in items]
    one = _slot_bytes(100_000)
    # all three wait in host memory but the first that fits: the queue's blocks
    # together never fit the budget
    ref, most = _run(host, budget=_slot_bytes(200_000) + 500)
    assert most == 1
    # all on the device from the start
    got, most = _run(host, budget=64 << 30)
    assert got == ref and most == 2
    # one slot: one block early, the others wait
    assert _run(host, budget=64 << 30, slots=1) == (ref, 1)
    # blocks 0 and 1 go early (they fit together), block 2 waits in host memory;
    # block 1 waits for its track and gives way to block 2
    budget = one + _slot_bytes(200_000) + 500
    assert 2 * one <= budget < one + _slot_bytes(200_000) + 100_000 * 4
    got, most = _run(host, budget=budget)
    assert got == ref and most == 2
    # samples in device memory; they may be overwritten after the submission
    dev = [torch.from_numpy(i["block"].samples).cuda() for _, i in items]
    srv = ptk.pt_server_create(ctx().handle, ptk.make_server_config(_settings(), max_slots=8, gens_per_step=32))
    try:
        order, out = {}, {}
        for k, (t, i) in enumerate(items):
            b = i["block"]
            blk = ptk.make_block(dev[k], b.fs, b.lo, b.hi, ref=b.ref, stream=b.stream)
            order[ptk.pt_server_submit(srv, t, blk)] = k
            dev[k].zero_()
        while len(out) < len(items):
            ptk.pt_server_step(srv, ptk.current_stream())
            for r in ptk.pt_server_poll(srv):
                out[order[r.ticket]] = _key(r)
        assert [out[k] for k in range(len(items))] == ref
    finally:
        ptk.pt_server_destroy(srv)


def test_buffers_pass_from_block_to_block():
    """Repeated streams of growing and shrinking blocks through one server."""
    items = _stream(ntracks=2, nblocks=4, seed=7)
    srv = ptk.pt_server_create(ctx().handle, ptk.make_server_config(_settings(), max_slots=3, gens_per_step=64))
    try:
        seen = []
        for rep in range(3):
            order, out = {}, {}
            for i in items if rep != 1 else items[::-1]:
                order[ptk.pt_server_submit(srv, 100 * rep + i["track"] * 10 + i["seq"], _blk(i))] = (i["track"], i["seq"])
            while len(out) < len(order):
                ptk.pt_server_step(srv, ptk.current_stream())
                for r in ptk.pt_server_poll(srv):
                    out[order[r.ticket]] = _key(r)
            seen.append(out)
        assert seen[0] == seen[1] == seen[2]
        assert all(np.isfinite(v).all() for v in seen[0].values())
    finally:
        ptk.pt_server_destroy(srv)
