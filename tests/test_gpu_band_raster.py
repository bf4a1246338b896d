"""The banded adjoint serves points that fill a wave inside a band where they stand (up to
width 8) and the others through the band's queue: the gradients of a point are the same
bits whichever way it comes, so those of points stored by rows equal those of the same
points in no order, at item sizes around the blocks the waves take in turn."""
import numpy as np
import pytest
import torch

import synth
from helpers import gpu_batch, make_plan

pytestmark = pytest.mark.gpu

COUNTS = [1, 63, 64, 65, 0, 511, 512, 513, 600, 2047, 2048, 2049, 9000]


@pytest.mark.parametrize("prec,eps,n_modes", [("f32", 1e-6, (64, 64)), ("f64", 1e-6, (64, 64)), ("f64", 1e-6, (33, 64)),
                                              ("f64", 1e-4, (64, 20)), ("f64", 1e-10, (64, 64))])
def test_rows_equal_no_order(prec, eps, n_modes):
    b = synth.uniform_box(counts=COUNTS, n_modes=n_modes, precision=prec, window_radius=3.0, seed=21)
    b.eps = eps
    gb = gpu_batch(b)
    plan = make_plan(gb)
    rng = np.random.default_rng(22)
    g = torch.as_tensor(rng.standard_normal((b.n_cells, n_modes[1], n_modes[0])) + 0.5j, device="cuda:0").to(plan.cdtype)
    off = np.asarray(b.cell_offsets)
    y = gb.y.cpu().numpy()
    perm = torch.as_tensor(np.concatenate([off[c] + np.argsort(y[off[c]:off[c + 1]], kind="stable")
                                           for c in range(b.n_cells)]), device="cuda:0")
    ref = plan.adjoint(gb.x, gb.y, gb.h, gb.w, g)
    got = plan.adjoint(*[v[perm].contiguous() for v in (gb.x, gb.y, gb.h, gb.w)], g)
    torch.cuda.synchronize()
    print(prec, eps, "W", plan.info()["kernel_width"], "bands", plan.info()["adj_bands"], flush=True)
    for r, t in zip(ref, got):
        assert torch.equal(r[perm], t)
