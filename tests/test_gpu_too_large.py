"""What is too large for the forms over the samples is refused whatever form it would take."""
import pytest
import torch

from gpu_util import ctx
from paper_1906_10598_amd import phasetrack as ptk

pytestmark = pytest.mark.gpu


@pytest.fixture
def one_row_units():
    ptk.pt_ctx_set_tile(ctx().handle, 4, 1)  # 1024 samples and one candidate in a work unit
    yield
    ptk.pt_ctx_set_tile(ctx().handle, 0, 0)


def _block(samples):
    return ptk.make_block(samples, 50_000.0, [0.6, 0.0, 1000.0, 0.0, 0.0, 0.0, 0.0], [0.8, 6.0, 1000.0005, 0.0, 0.0, 0.0, 0.0])


def test_batch_of_too_many_work_units(one_row_units):
    n = 1 << 26
    blk = _block(torch.zeros(n, dtype=torch.float32, device="cuda"))
    de = ptk.make_settings(pop=240, max_gens=1, F=0.5, CR=0.9, seed=1)
    units = (n // 1024) * 240
    blocks = [blk] * ((1 << 30) // units + 1)
    with pytest.raises(ptk.PtError, match="batch too large"):
        ctx().fit_batch(blocks, de)


def test_objective_of_too_many_work_units(one_row_units):
    n = (1 << 30) + 1024  # 2^20 + 1 tiles
    blk = _block(torch.zeros(n, dtype=torch.float32, device="cuda"))
    pop = torch.zeros(1024, ptk.NSLOT, dtype=torch.float64, device="cuda")
    with pytest.raises(ptk.PtError, match="batch too large"):
        ctx().objective(blk, pop)
    torch.cuda.empty_cache()
