"""The Voronoi search's edge cases: cells of one and two samples, exact duplicates
(ties go to the lowest index), all samples but one in one bin, sample counts around a
workgroup's rounds, and rasters below and above one round of listed centres."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_21278_amd as enf

pytestmark = pytest.mark.gpu

COUNTS = [1, 2, 15, 16, 17, 1023, 1024, 1025, 4097]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("raster", [1, 3, 32, 33, 70])
@pytest.mark.parametrize("mask", ["triangle", "circle"])
def test_search_edges(raster, mask, prec):
    rng = np.random.default_rng(raster)
    tri, xs, ys = [], [], []
    for i, n in enumerate(COUNTS):
        v = rng.uniform(-3, 3, (3, 2)) + rng.uniform(-20, 20, 2)
        tri.append(v.ravel())
        w = rng.dirichlet([1.0, 1.0, 1.0], n)
        p = w @ v
        if i % 3 == 1:      # all but the first at nearly one place
            p[1:] = p[0] + 1e-3 * rng.standard_normal((n - 1, 2))
        if i % 3 == 2:      # exact duplicates: every sample three times
            p = p[np.arange(n) // 3]
        xs.append(p[:, 0])
        ys.append(p[:, 1])
    dt = torch.float64 if prec == "f64" else torch.float32
    x, y = (torch.as_tensor(np.concatenate(v), device="cuda:0").to(dt) for v in (xs, ys))
    h = torch.as_tensor(rng.normal(100.0, 30.0, len(x)), device="cuda:0").to(dt)
    off = np.concatenate([[0], np.cumsum(COUNTS)])
    plan = enf.Plan(off, None, n_modes=(16, 16), precision=prec, window="none", eps=1e-5)
    kw = dict(frame="edge", mask=mask, weights="voronoi", raster=raster, eta=1.2)
    got = plan.cell_geometry(np.array(tri), x, y, h, need_counts=True, **kw)
    torch.cuda.synchronize()
    ref = oracle.cell_geometry(off, np.array(tri), *(t.cpu().double().numpy() for t in (x, y, h)), **kw)
    assert np.array_equal(got["inside"].cpu().numpy(), ref["inside"])
    assert np.array_equal(got["counts"].cpu().numpy(), ref["counts"])
    wb = got["wb"].cpu().double().numpy()
    # one rounding of the output type on FP64 sums taken in another order
    assert np.allclose(wb, ref["wb"], rtol=1e-13 if prec == "f64" else 6.1e-8, atol=0)
    # the same without the caller's counts (the workspace holds them)
    again = plan.cell_geometry(np.array(tri), x, y, h, need_counts=False, **kw)
    assert torch.equal(again["wb"], got["wb"]) and torch.equal(again["hb"], got["hb"])
