"""FP64 plans whose cells fit LDS evaluate kernel taps as polynomials.  Up to W = 8 these stand
for psi to a rounding error, the outermost pair in two parts split at psi's branch point:
type-1, adjoint and reconstruction agree with the same calls through psi itself
(ENUFFT_POLY64=0) in both oversampling regimes and with the Kaiser-Bessel kernel.  From
W = 10 one polynomial serves every tap, ten times and more below eps."""
import numpy as np
import pytest
import torch

import synth
from helpers import gpu_batch, make_plan, rel_l2

pytestmark = pytest.mark.gpu


def _outputs(gb, n_modes, monkeypatch, poly, **kw):
    monkeypatch.setenv("ENUFFT_POLY64", "1" if poly else "0")
    plan = make_plan(gb, **kw)
    rng = np.random.default_rng(12)
    g = torch.as_tensor(rng.standard_normal((gb.n_cells, n_modes[1], n_modes[0], 2)) @ np.array([1.0, 1j]),
                        device="cuda:0").contiguous()
    out = {"f": plan.type1(gb.x, gb.y, gb.h, gb.w)}
    out["gh"], out["gx"], out["gy"] = plan.adjoint(gb.x, gb.y, gb.h, gb.w, g)
    out["h_rec"], out["diag"] = plan.reconstruct(gb.x, gb.y, gb.h, gb.w, g)
    return plan.info(), {k: v.cpu().numpy() for k, v in out.items()}


@pytest.mark.parametrize("kernel", ["es", "kb_mirt"])
@pytest.mark.parametrize("sigma", [2.0, 1.5])
@pytest.mark.parametrize("eps", [1e-3, 1e-4, 1e-5, 1e-6, 1e-7, 1e-8, 1e-10])
def test_taps_equal_the_kernel(eps, sigma, kernel, monkeypatch):
    n_modes = (41, 20)
    b = synth.uniform_box(counts=[1, 65, 0, 1500], n_modes=n_modes, precision="f64", window_radius=3.0, seed=9)
    b.eps, b.sigma = eps, sigma
    gb = gpu_batch(b)
    info, got = _outputs(gb, n_modes, monkeypatch, True, kernel=kernel)
    _, ref = _outputs(gb, n_modes, monkeypatch, False, kernel=kernel)
    print(eps, sigma, kernel, "W", info["kernel_width"], "fit %.1e" % info["kernel_poly_err"],
          {k: "%.1e" % rel_l2(got[k], ref[k]) for k in got}, flush=True)
    assert info["kernel_poly_err"] <= (1e-13 if info["kernel_width"] <= 8 else 0.1 * eps)
    # a footprint's two axes deviate by that much of psi's peak each, about 4.5 times as much
    # of its norm; deconvolution weighs the edge of the box up to 20 times its centre
    for k in got:
        assert rel_l2(got[k], ref[k]) <= 100 * (info["kernel_poly_err"] + 2.0 ** -52), k
