"""Bare evaluations on both sides of the size from which the fits' objective kernels
run them: the same rows give the same bits, and the oracle's values."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import assert_chi2_close, block_of, ctx, model_phase_err, random_population, to_dev
from paper_1906_10598_amd import phasetrack as ptk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("objective", [ptk.PT_OBJ_CHI2, ptk.PT_OBJ_COR])
@pytest.mark.parametrize("precision,n", [(ptk.PT_PREC_FP64, 1_050_001), (ptk.PT_PREC_MIXED, 650_003)])
@pytest.mark.parametrize("slot,value", [(None, 0.0), (5, 0.01), (6, 1e-4), (2, 0.0), (3, np.nan)])
def test_the_same_rows_on_both_sides(slot, value, precision, n, objective):
    b = synth.config1(3, n=n)
    if precision == ptk.PT_PREC_FP64 and objective == ptk.PT_OBJ_CHI2:
        b.samples = b.samples.astype(np.float64)
    dev = to_dev(b.samples)
    blk = block_of(b, dev)
    pop = random_population(np.random.default_rng(7), b.lo, b.hi, 270)
    pop[:, 5:] = 0.0
    if slot is not None:
        pop[111, slot] = value
    more = np.concatenate([pop, pop[:30]])  # (one tile sum after the other in both: P > 256)
    assert 270 * n < (1.9e8 if precision == ptk.PT_PREC_MIXED else 3e8) <= 300 * n
    c = ctx()
    ptk.pt_ctx_set_tile(c.handle, 32, 8)
    try:
        below = c.objective(blk, to_dev(pop), precision, objective).cpu().numpy()
        arith = ptk.pt_ctx_last_arithmetic(c.handle)
        above = c.objective(blk, to_dev(more), precision, objective).cpu().numpy()
        assert ptk.pt_ctx_last_arithmetic(c.handle) == arith
        assert ptk.pt_ctx_last_geometry(c.handle) == (32, 8)
        assert np.array_equal(above[:270], below, equal_nan=True)
        assert np.array_equal(above[270:], below[:30], equal_nan=True)
        d_pop, out = to_dev(more), to_dev(np.zeros(300))
        ptk.pt_objective_noalloc(c.handle, blk, d_pop.data_ptr(), 300, precision, out.data_ptr(), objective=objective)
        assert np.array_equal(out.cpu().numpy(), above, equal_nan=True)
        if precision == ptk.PT_PREC_FP64 and objective == ptk.PT_OBJ_CHI2:
            idx = [0, 110, 269]
            want = oracle.chi2_pop(b.samples, b.fs, b.ref, pop[idx])
            assert_chi2_close(above[idx], want, n, amp=float(np.max(pop[:, 0])), floor=model_phase_err(c))
    finally:
        ptk.pt_ctx_set_tile(c.handle, 0, 0)
