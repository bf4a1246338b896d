"""FP64 large cells on the matrix cores: every kernel width they serve (and one beyond),
at point counts around the padding of a block and a round of points, with points at
the tile and grid edges, all in one fine cell, and clustered.  Type-1 and the analytic
VJP against the oracle's direct sums."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2606_21278_amd as enf
from helpers import rel_l2

pytestmark = pytest.mark.gpu


def _points(kind, n, rng, cells):
    d = 2 * math.pi / cells
    if kind == "edges":      # on and beside tile boundaries and the wrap of the box
        x = (rng.integers(-cells // 32, cells // 32 + 1, n) * 32 + rng.integers(-3, 4, n) + 0.5 * rng.random(n)) * d
        y = (rng.integers(-cells // 32, cells // 32 + 1, n) * 32 + rng.integers(-3, 4, n) + 0.5 * rng.random(n)) * d
    elif kind == "cell":     # one fine cell
        x, y = 1.0 + 0.4 * d * rng.random(n), -2.0 + 0.4 * d * rng.random(n)
    else:                    # background and a cluster
        x, y = rng.uniform(-math.pi, math.pi, (2, n))
        m = n // 2
        x[:m], y[:m] = 0.5 + 0.05 * rng.standard_normal(m), -1.0 + 0.05 * rng.standard_normal(m)
    return x, y


@pytest.mark.parametrize("eps", [1e-3, 1e-5, 1e-7, 1e-9, 1e-11, 1e-12])
@pytest.mark.parametrize("kind,n", [("mixed", 1), ("mixed", 17), ("edges", 1500), ("cell", 700), ("mixed", 9001)])
def test_fp64_large_cells(kind, n, eps):
    rng = np.random.default_rng(n)
    x, y = _points(kind, n, rng, 256)
    h, w = rng.standard_normal(n), rng.uniform(0.5, 1.5, n)
    win = np.array([[0.0, 0.0, 6.0]])
    plan = enf.Plan([0, n], win, n_modes=(90, 72), precision="f64", eps=eps)
    t = [torch.as_tensor(v, dtype=torch.float64, device="cuda:0") for v in (x, y, h, w)]
    f = plan.type1(*t).cpu().numpy()
    ref = oracle.type1([0, n], x, y, h, w, win, (90, 72))
    g = rng.standard_normal((1, 72, 90)) + 1j * rng.standard_normal((1, 72, 90))
    grads = plan.adjoint(*t, torch.as_tensor(g, device="cuda:0"))
    rgrads = oracle.type1_vjp([0, n], x, y, h, w, win, (90, 72), g)
    errs = [rel_l2(f, ref)] + [rel_l2(a.cpu().numpy(), b) for a, b in zip(grads, rgrads)]
    print(kind, n, eps, "W", plan.info()["kernel_width"], errs, flush=True)
    # the kernel's truncation error is of the order of eps, larger for a lone point's
    # few values; rounding of the sums on top
    assert max(errs) <= 20 * eps + 1e-12
