"""Device memory that a server keeps between blocks stays within its budget."""
import pytest
import torch

from gpu_util import ctx
from paper_1906_10598_amd import phasetrack as ptk

pytestmark = pytest.mark.gpu

MIB = 1 << 20


def _free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


@pytest.mark.parametrize("on_device", [True, False])
@pytest.mark.parametrize("growing", [True, False])
def test_blocks_of_many_sizes(growing, on_device):
    """Blocks of 32 to 64 MiB one after the other (each needs another buffer than the
    last, or passes its own on), then two at a time, in a budget of 1.2 of the largest."""
    sizes = [(32 + 8 * k) * MIB // 4 for k in range(5)]
    if not growing:
        sizes = sizes[::-1]
    fs, x = 50_000.0, [0.7, 1.3, 1234.5, 0.0, 0.0, 0.0, 0.0]
    half = [0.1, 3.0, 1e-3, 0.0, 0.0, 0.0, 0.0]
    lo, hi = [a - h for a, h in zip(x, half)], [a + h for a, h in zip(x, half)]
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    samples = []
    for n in sizes:
        t = (torch.arange(n, dtype=torch.float64, device="cuda") - n / 2) / fs
        s = 0.7 * torch.cos(1.3 + 2 * torch.pi * torch.frac(1234.5 * t))
        s += 0.4 * torch.randn(n, generator=g, device="cuda", dtype=torch.float64)
        samples.append(s.float() if on_device else s.float().cpu())
        del t, s
    torch.cuda.empty_cache()
    de = ptk.make_settings(pop=8, max_gens=20, F=0.5, CR=0.9, seed=1)
    # (what the runtime takes when kernels run for the first time is none of the server's)
    first = ptk.pt_server_create(ctx().handle, ptk.make_server_config(de, max_slots=1, gens_per_step=32))
    ptk.pt_server_submit(first, 0, ptk.make_block(samples[0], fs, lo, hi))
    ptk.pt_server_step(first, ptk.current_stream())
    ptk.pt_server_destroy(first)
    budget = int(1.2 * 64 * MIB)
    srv = ptk.pt_server_create(ctx().handle, ptk.make_server_config(de, max_slots=4, gens_per_step=32,
                                                                    hbm_budget_bytes=budget))
    try:
        before, most = _free(), 0
        track = 0
        for group in [[s] for s in samples] + [samples[:2], samples[3:]]:
            for s in group:
                ptk.pt_server_submit(srv, track, ptk.make_block(s, fs, lo, hi, stream=track))
                track += 1
                most = max(most, before - _free())
            left = len(group)
            while left:
                ptk.pt_server_step(srv, ptk.current_stream())
                left -= len(ptk.pt_server_poll(srv))
                most = max(most, before - _free())
        print(f"[server memory growing {growing}] {most / MIB:.0f} of {budget / MIB:.0f} MiB", flush=True)
        # what the budget does not count (weights, draws, working space: 1024 tiles of 2 KiB
        # and 128 groups of moments at most) and the rounding of a dozen allocations to 2 MiB
        assert most <= budget + 32 * MIB
    finally:
        ptk.pt_server_destroy(srv)
