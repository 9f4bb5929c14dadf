"""The rule that keeps fits of a few generations on many nodes over their samples:
on the host against measured fits, and on the device its route."""
import ctypes
import subprocess

import numpy as np
import pytest

import synth
from paper_1906_10598_amd import build

SOURCE = """
#include "nodes.h"
extern "C" int pays(int K, long long n, int P, int max_gens) { return pt::node_pays(K, n, P, max_gens); }
"""

# nodes, samples, members, generations; microseconds of a fit through nodes and over its samples
MEASURED = [(464, 50_000, 8, 1, 156, 56), (464, 50_000, 8, 20, 257, 154), (464, 50_000, 8, 100, 355, 611),
            (464, 50_000, 40, 1, 101, 56), (464, 50_000, 40, 20, 266, 191), (464, 50_000, 40, 100, 536, 784),
            (464, 400_000, 40, 1, 104, 80), (464, 400_000, 40, 20, 269, 416), (464, 400_000, 240, 20, 801, 1468),
            (464, 50_000, 240, 20, 789, 412), (464, 50_000, 240, 500, 1928, 8182),
            (256, 4096, 240, 1, 98, 52), (256, 4096, 240, 20, 482, 203), (256, 4096, 240, 100, 906, 797),
            (256, 4096, 240, 500, 1415, 3692), (256, 400_000, 8, 1, 85, 56), (256, 400_000, 8, 20, 148, 235),
            (256, 50_000, 120, 1, 75, 65), (112, 4096, 240, 20, 276, 203), (112, 4096, 240, 100, 530, 798),
            (112, 4096, 40, 20, 97, 147), (112, 400_000, 240, 1, 79, 208), (48, 512, 240, 1, 65, 50),
            (48, 512, 8, 20, 64, 152), (48, 4096, 120, 20, 109, 171), (48, 400_000, 40, 1, 52, 81),
            (48, 400_000, 40, 500, 269, 7955)]


@pytest.fixture(scope="module")
def pays(tmp_path_factory):
    d = tmp_path_factory.mktemp("node_pays")
    src, lib = d / "host.hip", d / "libhost.so"
    src.write_text(SOURCE)
    subprocess.run(["/opt/rocm/bin/hipcc", *build.HIPCC_FLAGS, f"-I{build.CSRC}", "-shared", str(src), "-o", str(lib)],
                   check=True, stderr=subprocess.DEVNULL)
    f = ctypes.CDLL(str(lib)).pays
    f.argtypes = [ctypes.c_int, ctypes.c_longlong, ctypes.c_int, ctypes.c_int]
    return f


def test_the_faster_route_of_measured_fits(pays):
    for K, n, P, gens, nodes, samples in MEASURED:
        assert bool(pays(K, n, P, gens)) == (nodes < samples), (K, n, P, gens)


def test_longer_fits_on_fewer_nodes_stay(pays):
    # more generations (past the few that two or three differ by) and fewer nodes never turn it round
    for n in (64, 4096, 400_000, 1 << 26):
        for P in (4, 40, 57, 121, 240):
            row = [[pays(K, n, P, g) for g in (0, 40, 400, 1500, 1 << 30)] for K in (16, 64, 256, 512)]
            assert all(r[k] <= r[k + 1] for r in row for k in range(1, 4)) and all(r[3] for r in row)
            assert all(a[k] >= b[k] for a, b in zip(row, row[1:]) for k in range(5))


@pytest.mark.gpu
@pytest.mark.parametrize("gens,nodes", [(3, False), (400, True)])
def test_short_fits_of_wide_boxes_run_over_their_samples(gens, nodes):
    from gpu_util import block_of, ctx, settings_of, to_dev
    from paper_1906_10598_amd import phasetrack as ptk
    from test_gpu_nodes import _block, _fit, _same

    b = _block(50_000, half=(0.1, 3.0, 60.0, 0.0, 0.0, 0.0, 0.0))
    pb = block_of(b, to_dev(b.samples))
    de = settings_of(b, gens=gens)
    a = _fit([pb], de)
    assert (ptk.pt_ctx_fit_launches(ctx().handle) == 1) == nodes
    g = _fit([pb], de, ptk.PT_LAUNCH_GRAPH)
    if not nodes:
        _same(a, g)
    # served, alone and in a batch alike
    srv = ptk.pt_server_create(ctx().handle, ptk.make_server_config(de, max_slots=2, gens_per_step=8, spl=16, cpg=8))
    ptk.pt_ctx_set_tile(ctx().handle, 16, 8)
    try:
        small = block_of(synth.config1(0, n=50_000), to_dev(synth.config1(0, n=50_000).samples))
        alone, both = _fit([pb], de), _fit([pb, small], de)
        ptk.pt_server_submit(srv, 0, pb)
        got = []
        while not got:
            ptk.pt_server_step(srv, ptk.current_stream())
            got = ptk.pt_server_poll(srv)
        for f in (both[0][0], got[0].fit):
            assert list(f.coef) == list(alone[0][0].coef) and f.objective == alone[0][0].objective
    finally:
        ptk.pt_ctx_set_tile(ctx().handle, 0, 0)
        ptk.pt_server_destroy(srv)
    assert np.isfinite(a[0][0].objective)
