"""Tests of the launch forms that evaluate every sample, with those forms pinned.

In the automatic launch mode most fits go through node weights, which have one
form: there a comparison of step fusions compares a fit with itself.  Here the
same tests run with PT_LAUNCH_GRAPH, and every fit is seen to take a launch or
more per generation.
"""
import pytest

from gpu_util import ctx
from paper_1906_10598_amd import phasetrack as ptk
from test_gpu_fit import (test_amplitude_slope_fit_matches_oracle, test_batch_equals_alone,  # noqa: F401
                          test_batch_splits_blocks_by_arithmetic, test_host_samples_match_device_samples,
                          test_tiny_block_fit_matches_oracle, test_truth_outside_box_flags_at_bound,
                          test_window_rule_and_vtr_match_oracle)
from test_gpu_fusion import (test_batch_with_window_rule, test_graph_cache_eviction_keeps_fits_bitwise,  # noqa: F401
                             test_paper_block, test_populations_past_one_wave, test_short_windows,
                             test_stop_at_generation_zero_and_no_generations, test_timed_fit_equals_two_launch_form,
                             test_tiny_block)
from test_gpu_server import test_leading_step_server_equals_default, test_warm_start_tracks_the_phase  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def over_the_samples(monkeypatch):
    c = ctx()
    create, block, batch = ptk.Context.__init__, ptk.Context.fit_block, ptk.Context.fit_batch

    def created(self, *a, **kw):
        create(self, *a, **kw)
        ptk.pt_ctx_set_launch_mode(self.handle, ptk.PT_LAUNCH_GRAPH)

    def fit_block(self, *a, **kw):
        f = block(self, *a, **kw)
        assert ptk.pt_ctx_fit_launches(self.handle) >= f.generations + 1
        return f

    def fit_batch(self, *a, **kw):
        fits = batch(self, *a, **kw)
        assert ptk.pt_ctx_fit_launches(self.handle) >= max(f.generations for f in fits) + 1
        return fits

    monkeypatch.setattr(ptk.Context, "__init__", created)
    monkeypatch.setattr(ptk.Context, "fit_block", fit_block)
    monkeypatch.setattr(ptk.Context, "fit_batch", fit_batch)
    ptk.pt_ctx_set_launch_mode(c.handle, ptk.PT_LAUNCH_GRAPH)
    yield
    ptk.pt_ctx_set_launch_mode(c.handle, ptk.PT_LAUNCH_AUTO)
