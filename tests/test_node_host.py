"""Host side of the node-weight fits that needs no GPU: what nodes.h says about
draws and launches, through a small library built from that header."""
import ctypes
import subprocess

import pytest

from paper_1906_10598_amd import build

SOURCE = """
#include "nodes.h"
extern "C" {
size_t draw_words(int P, int gens) { return pt::node_draw_words(P, gens); }
int octet_members(int P) { return pt::node_nm(P); }
int member_waves(int P) { return pt::node_waves(P); }
}
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("node_host")
    src, lib = d / "host.hip", d / "libhost.so"
    src.write_text(SOURCE)
    subprocess.run(["/opt/rocm/bin/hipcc", *build.HIPCC_FLAGS, f"-I{build.CSRC}", "-shared", str(src), "-o", str(lib)],
                   check=True, stderr=subprocess.DEVNULL)
    so = ctypes.CDLL(str(lib))
    so.draw_words.restype = ctypes.c_size_t
    return so


def test_draws_of_any_stretch_of_generations(host):
    """The place holds the blocks of 16 generations that a launch touches wherever it
    begins, 128 words per wave and member of its octets each -- and no generations
    take none, so the last launch of a fit starts no workgroups to draw them."""
    for P in (4, 40, 120, 121, 240):
        per = 128 * host.octet_members(P) * host.member_waves(P)
        assert host.draw_words(P, 0) == 0
        for gens in (1, 2, 15, 16, 17, 512, 2048):
            blocks = max((g0 + gens - 1) // 16 - g0 // 16 + 1 for g0 in range(32))
            assert host.draw_words(P, gens) == blocks * per
