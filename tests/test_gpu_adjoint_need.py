"""The adjoint asked for some of its gradients equals the same gradients of the full
call: the single-grid adjoint (FP32) and the banded one (FP64), point counts around a
wave's and a workgroup's."""
import numpy as np
import pytest
import torch

import synth
from helpers import gpu_batch, make_plan, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("need", [(True, False, False), (False, True, False), (False, False, True), (True, False, True),
                                  (False, True, True)])
def test_some_gradients_equal_the_full_call(prec, need):
    b = synth.uniform_box(counts=[1, 63, 64, 65, 0, 511, 512, 513, 2001], n_modes=(64, 64), precision=prec,
                          window_radius=3.0, seed=13)
    gb = gpu_batch(b)
    plan = make_plan(gb)
    rng = np.random.default_rng(14)
    g = rng.standard_normal((b.n_cells, 64, 64, 2)) @ np.array([1.0, 1j])
    g = torch.as_tensor(g, device="cuda:0").to(plan.cdtype).contiguous()
    full = plan.adjoint(gb.x, gb.y, gb.h, gb.w, g)
    some = plan.adjoint(gb.x, gb.y, gb.h, gb.w, g, need=need)
    for on, s, f in zip(need, some, full):
        assert (s is not None) == on
        if on:   # the same sums; the two builds may contract a product and a sum differently
            assert rel_l2(s.cpu().numpy(), f.cpu().numpy()) <= 16 * (2.0 ** -24 if prec == "f32" else 2.0 ** -53)
