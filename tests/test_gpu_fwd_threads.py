"""The forward's workgroup size by the plan's cells and points: both sides of the rule,
and the same coefficients from either size."""
import pytest
import torch

import synth
from helpers import gpu_batch, make_plan, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("below", ["none", "cells", "points"])
def test_forward_threads_rule(below, monkeypatch):
    n = 8 * torch.cuda.get_device_properties(0).multi_processor_count - (below == "cells")
    counts = [8191 + 2 * (c % 2) for c in range(n)]
    counts[0] += sum(8192 - q for q in counts) - (below == "points")
    b = synth.uniform_box(counts=counts, n_modes=(64, 64), precision="f32", window_radius=3.0, seed=2)
    gb = gpu_batch(b)
    plan = make_plan(gb)
    assert plan.info()["kernel_width"] <= 6
    assert plan.info()["fwd_threads"] == (1024 if below == "none" else 512)
    got = plan.type1(gb.x, gb.y, gb.h, gb.w).cpu().numpy()
    monkeypatch.setenv("ENUFFT_FWD_THREADS", "512")
    ref = make_plan(gb).type1(gb.x, gb.y, gb.h, gb.w).cpu().numpy()
    # the same FP64 sums in another order, rounded once to FP32: a unit in the last place
    # of a few grid values
    assert rel_l2(got, ref) <= 2.0 ** -23
