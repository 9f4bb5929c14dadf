"""Node-weight fits longer than one launch: 2048 generations, 512 with the window
rule.  Bit for bit the fits of one generation a launch (timing)."""
import pytest

import synth
from gpu_util import block_of, ctx, settings_of, to_dev
from paper_1906_10598_amd import phasetrack as ptk
from test_gpu_nodes import _fit, _same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pop", [32, 130])
@pytest.mark.parametrize("gens,window,launches", [(2046, False, 1), (2047, False, 1), (2048, False, 2), (2049, False, 2),
                                                  (4200, False, 3), (511, True, 1), (512, True, 2), (1300, True, 3)])
def test_launches_of_a_long_fit(pop, gens, window, launches):
    b = synth.config0(3)
    pb = block_of(b, to_dev(b.samples))
    # (a window longer than the fit: the rule is on and never met)
    de = settings_of(b, gens=gens, pop=pop, **(dict(rel_tol=1e-300, window=gens + 1) if window else {}))
    a = _fit([pb], de)
    assert ptk.pt_ctx_fit_launches(ctx().handle) == launches
    t = _fit([pb], de, timing=True)
    assert ptk.pt_ctx_fit_launches(ctx().handle) == gens + 1
    _same(a, t)
    assert a[0][0].generations == gens and len(a[0][3]) == gens + 1
