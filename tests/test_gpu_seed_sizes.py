"""Every snippet size of the seeding spectrum, with the peak in its middle and
in its first and last usable bins (odd and even log2: the transform begins
with a radix-2 or a radix-4 pass).  Oracle and tolerances: test_gpu_seed.
"""
import numpy as np
import pytest

import synth
from gpu_util import ctx
from paper_1906_10598_amd import phasetrack as ptk
from test_gpu_seed import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("log", range(6, 14))
def test_every_size_and_edge_bin(log, dtype):
    M = 1 << log
    if M > ptk.pt_seed_max_snippet(ctx().handle):
        pytest.skip("larger than this device's snippets")
    b = synth.config1(2, n=3 * M + 1)
    g = np.random.default_rng(log)
    t = np.arange(b.n)
    for bin_ in (1.3, M / 2 - 1.3, 0.37 * M):
        s = np.cos(2 * np.pi * bin_ / M * t + 1.0) + 0.1 * g.standard_normal(b.n)
        # an odd first sample for the centre snippet, spacing not a multiple of four
        r, _ = _check(b, M, spacing=M - 1, samples=s.astype(dtype))
        assert abs(r.bin[1] - bin_) <= 1
