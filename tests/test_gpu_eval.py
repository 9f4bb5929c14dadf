"""Bare objective evaluations whose arithmetic the device chooses from the rows.

The kernel takes the rows' extents itself (slope, quartic term, the FP64 phasor
path's bounds), so one row anywhere has to decide for all; the workgroup that
finishes last adds up the tiles' sums for populations of up to 256 members, a
second launch for larger ones.  Oracle and tolerances are those of
test_gpu_objective.
"""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import assert_chi2_close, block_of, ctx, model_phase_err, random_population, to_dev
from paper_1906_10598_amd import phasetrack as ptk

pytestmark = pytest.mark.gpu

N = 20_011  # five ragged tiles of 4096 samples


@pytest.mark.parametrize("P", [1, 2, 5, 64, 65, 255, 256, 257, 1024])
def test_one_row_decides_for_all(P):
    b = synth.config1(1, n=N)
    dev = to_dev(b.samples)
    blk = block_of(b, dev)
    s = b.samples.astype(np.float64)
    base = random_population(np.random.default_rng(P), b.lo, b.hi, P)
    base[:, 5:] = 0.0
    amp = float(np.max(np.abs(base[:, 0])))
    c = ctx()
    ptk.pt_ctx_set_tile(c.handle, 16, 4)  # the phasor path's bounds hold for the box
    try:
        # (slot, value of the last row, the arithmetic it leaves to all rows):
        # a slope (20 % of the amplitude over the block), a quartic term of half
        # a turn at the ends, a carrier at 0 Hz (the recurrence would not hold)
        th = 0.5 * N / b.fs
        for slot, value, want_arith in [(None, 0.0, ptk.PT_ARITH_FP64_PHASOR),
                                        (5, 0.4 * b.fs / N, ptk.PT_ARITH_FP64_PHASOR),
                                        (6, 12.0 / th ** 4, None),
                                        (2, 0.0, ptk.PT_ARITH_FP64_POLY),
                                        (None, 0.0, ptk.PT_ARITH_FP64_PHASOR)]:
            pop = base.copy()
            if slot is not None:
                pop[-1, slot] = value
            got = c.objective(blk, to_dev(pop), ptk.PT_PREC_FP64).cpu().numpy()
            arith = ptk.pt_ctx_last_arithmetic(c.handle)
            assert want_arith is None or arith == want_arith, (slot, arith)
            want = oracle.chi2_pop(s, b.fs, b.ref, pop)
            assert_chi2_close(got, want, N, amp=amp, floor=model_phase_err(c))
            again = c.objective(blk, to_dev(pop), ptk.PT_PREC_FP64).cpu().numpy()
            assert np.array_equal(got, again)
            # the allocation-free entry point: other launches, the same bits
            d_pop, out = to_dev(pop), to_dev(np.zeros(P))
            ptk.pt_objective_noalloc(c.handle, blk, d_pop.data_ptr(), P, ptk.PT_PREC_FP64, out.data_ptr())
            assert np.array_equal(got, out.cpu().numpy())
    finally:
        ptk.pt_ctx_set_tile(c.handle, 0, 0)


def test_a_row_that_is_not_a_number_spoils_only_itself():
    b = synth.config1(2, n=N)
    dev = to_dev(b.samples)
    pop = random_population(np.random.default_rng(3), b.lo, b.hi, 70)
    pop[:, 5:] = 0.0
    want = oracle.chi2_pop(b.samples.astype(np.float64), b.fs, b.ref, pop)
    for slot in range(7):
        q = pop.copy()
        q[33, slot] = np.nan
        got = ctx().objective(block_of(b, dev), to_dev(q), ptk.PT_PREC_FP64).cpu().numpy()
        assert np.isnan(got[33])
        rest = np.arange(70) != 33
        assert_chi2_close(got[rest], want[rest], N, amp=float(np.max(np.abs(pop[:, 0]))), floor=model_phase_err())
