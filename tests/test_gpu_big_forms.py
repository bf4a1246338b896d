"""FP64 large cells run their unit passes on the matrix cores or one point per lane, by the
points per tile: both forms (ENUFFT_M64_PER_TILE) give the same coefficients and gradients
at point counts around a block's padding, a round of points and the rule's line."""
import math

import numpy as np
import pytest
import torch

import paper_2606_21278_amd as enf
from helpers import rel_l2

pytestmark = pytest.mark.gpu


def _points(kind, n, rng, cells):
    d = 2 * math.pi / cells
    if kind == "edges":      # on and beside tile boundaries and the wrap of the box
        x, y = ((rng.integers(-cells // 32, cells // 32 + 1, n) * 32 + rng.integers(-3, 4, n) + 0.5 * rng.random(n)) * d
                for _ in range(2))
    elif kind == "cell":     # one fine cell
        x, y = 1.0 + 0.4 * d * rng.random(n), -2.0 + 0.4 * d * rng.random(n)
    else:                    # background and a cluster
        x, y = rng.uniform(-math.pi, math.pi, (2, n))
        m = n // 2
        x[:m], y[:m] = 0.5 + 0.05 * rng.standard_normal(m), -1.0 + 0.05 * rng.standard_normal(m)
    return x, y


@pytest.mark.parametrize("eps", [1e-5, 1e-7, 1e-9, 1e-11, 1e-12])   # W = 6 .. 14
@pytest.mark.parametrize("kind,n", [("mixed", 1), ("mixed", 17), ("edges", 1500), ("cell", 700), ("mixed", 6143),
                                    ("mixed", 6144), ("mixed", 9001)])
def test_forms_agree(kind, n, eps, monkeypatch):
    rng = np.random.default_rng(n)
    x, y = _points(kind, n, rng, 256)
    h, w = rng.standard_normal(n), rng.uniform(0.5, 1.5, n)
    g = rng.standard_normal((1, 72, 90)) + 1j * rng.standard_normal((1, 72, 90))
    t = [torch.as_tensor(v, dtype=torch.float64, device="cuda:0") for v in (x, y, h, w)]
    out = {}
    for per_tile in ("0", "1e18", None):   # 64 tiles: the line is at 6,144 points
        if per_tile is None:
            monkeypatch.delenv("ENUFFT_M64_PER_TILE")
        else:
            monkeypatch.setenv("ENUFFT_M64_PER_TILE", per_tile)
        plan = enf.Plan([0, n], np.array([[0.0, 0.0, 6.0]]), n_modes=(90, 72), precision="f64", eps=eps)
        f = plan.type1(*t)
        out[per_tile] = [f.cpu().numpy()] + [v.cpu().numpy() for v in plan.adjoint(*t, torch.as_tensor(g, device="cuda:0"))]
    # the same taps and FP64 sums in another order
    for form in ("0", None):
        errs = [rel_l2(a, b) for a, b in zip(out[form], out["1e18"])]
        assert max(errs) <= 1e-12, (form, errs)
