"""FP64 spreading and gathering four points at a time (one per row of sixteen lanes) at
every width they serve: point counts around the rounds of 4, 16, 64 and 512, footprints
that wrap the grid, and points outside the cell window, against the oracle's direct sums
and its analytic VJP."""
import numpy as np
import pytest
import torch

import oracle
import synth
from helpers import gpu_batch, make_plan, oracle_f, per_cell_rel_l2, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps,width,n_modes", [(1e-8, 10, (64, 64)), (1e-10, 12, (64, 64)), (1e-10, 12, (16, 9)),
                                               (1e-12, 14, (33, 20)), (1e-13, 16, (64, 64))])
def test_row_spread_counts(eps, width, n_modes):
    b = synth.uniform_box(counts=[1, 3, 4, 15, 17, 63, 65, 0, 511, 513, 3001], n_modes=n_modes, precision="f64",
                          window_radius=2.9, seed=5)
    b.eps = eps
    gb = gpu_batch(b)
    plan = make_plan(gb, kernel_width=width)
    assert plan.info()["kernel_width"] == width
    got = plan.type1(gb.x, gb.y, gb.h, gb.w).cpu().numpy()
    e = per_cell_rel_l2(got, oracle_f(b))
    print(eps, n_modes, np.nanmax(e), flush=True)
    # the kernel's truncation error is of the order of eps (1e-13: rounding of the grid
    # transforms on top); a cell of few points outside the window is exactly zero
    assert np.nanmax(e) <= 5 * eps + 1e-12


@pytest.mark.parametrize("eps,width,n_modes", [(1e-8, 10, (64, 64)), (1e-10, 12, (16, 9)), (1e-12, 14, (33, 20)),
                                               (1e-13, 16, (64, 64))])
def test_row_gather_counts(eps, width, n_modes):
    b = synth.uniform_box(counts=[1, 3, 4, 15, 17, 63, 65, 0, 511, 513, 3001], n_modes=n_modes, precision="f64",
                          window_radius=2.9, seed=8)
    b.eps = eps
    gb = gpu_batch(b)
    plan = make_plan(gb, kernel_width=width)
    rng = np.random.default_rng(9)
    g = rng.standard_normal((b.n_cells, n_modes[1], n_modes[0], 2)) @ np.array([1.0, 1j])
    got = plan.adjoint(gb.x, gb.y, gb.h, gb.w, torch.as_tensor(g, device="cuda:0").to(plan.cdtype).contiguous())
    inp = oracle.batch_inputs(b)
    ref = oracle.type1_vjp(inp["offsets"], inp["x"], inp["y"], inp["h"], inp["w"], inp["windows"], inp["n_modes"], g,
                           kind=inp["kind"])
    errs = [rel_l2(t.cpu().numpy(), r) for t, r in zip(got, ref)]
    print(eps, n_modes, errs, flush=True)
    assert max(errs) <= 5 * eps + 1e-12
