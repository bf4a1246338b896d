"""The banded adjoint (FP64 plans, and FP32 kernels of width 8): column spectra
transformed once per cell, row bands built from them, the points of each band queued
and gathered 64 at a time.  Against the oracle's analytic VJP at the band edges, odd
point counts and every kernel width, and across the groups of cells whose column
spectra are held at once."""
import numpy as np
import pytest
import torch

import oracle
import synth
from helpers import gpu_batch, make_plan, rel_l2

pytestmark = pytest.mark.gpu


def _vjp(b, plan, gb, g, cells):
    gg = torch.as_tensor(g, device="cuda:0").to(plan.cdtype).contiguous()
    got = plan.adjoint(gb.x, gb.y, gb.h, gb.w, gg)
    torch.cuda.synchronize()
    inp = oracle.batch_inputs(b.to(dtype=gb.x.dtype), cells)
    gc = gg.cpu().numpy().astype(np.complex128)[cells]
    ref = oracle.type1_vjp(inp["offsets"], inp["x"], inp["y"], inp["h"], inp["w"], inp["windows"], inp["n_modes"], gc,
                           kind=inp["kind"])
    off = np.asarray(b.cell_offsets)
    idx = np.concatenate([np.arange(off[c], off[c + 1]) for c in cells])
    return [rel_l2(t.cpu().numpy()[idx], r) for t, r in zip(got, ref)]


@pytest.mark.parametrize("prec,eps,n_modes", [("f64", 1e-7, (64, 64)), ("f64", 1e-9, (64, 64)), ("f64", 1e-10, (64, 64)),
                                              ("f64", 1e-12, (64, 64)), ("f64", 1e-13, (64, 64)),
                                              ("f64", 1e-10, (17, 9)), ("f64", 1e-10, (8, 64)),
                                              ("f32", 1e-6, (64, 64)), ("f32", 1e-6, (33, 20))])
def test_band_adjoint_widths_and_counts(prec, eps, n_modes):
    b = synth.uniform_box(counts=[1, 63, 64, 65, 0, 700, 3001], n_modes=n_modes, precision=prec, window_radius=3.0,
                          seed=3)
    b.eps = eps
    gb = gpu_batch(b)
    plan = make_plan(gb)
    rng = np.random.default_rng(4)
    g = rng.standard_normal((b.n_cells, n_modes[1], n_modes[0], 2)) @ np.array([1.0, 1j])
    errs = _vjp(b, plan, gb, g, list(range(b.n_cells)))
    print(prec, eps, n_modes, "W", plan.info()["kernel_width"], "bands", plan.info()["adj_bands"], errs, flush=True)
    # the kernel's truncation error is of the order of eps on every gradient (FP32: the
    # library's stated 5e-5; FP64 at 1e-13: the rounding of 64 x 64 modes on top)
    assert max(errs) <= (5e-5 if prec == "f32" else 5 * eps + 1e-12)


def test_band_adjoint_cell_groups():
    """Enough FP64 cells that their column spectra (270 KB each) take two groups."""
    n = 2100
    b = synth.uniform_box(counts=[3 + c % 5 for c in range(n)], n_modes=(64, 64), precision="f64", window_radius=3.0,
                          seed=6)
    gb = gpu_batch(b)
    plan = make_plan(gb)
    rng = np.random.default_rng(7)
    g = rng.standard_normal((n, 64, 64)) + 1j * rng.standard_normal((n, 64, 64))
    errs = _vjp(b, plan, gb, g, [0, 1, 1980, 1981, 1982, 1983, 1984, 1985, 1986, 1987, 1988, 1989, 1990, n - 1])
    print(errs, flush=True)
    assert max(errs) <= 5e-10
