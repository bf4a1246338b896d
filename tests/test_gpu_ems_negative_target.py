"""A target alpha_C below zero: alpha_min > alpha_max with w1 + w2 > 1 passes the parameter
checks (each is bounded by itself) and puts alpha_C = alpha_min + (alpha_max - alpha_min) C
below zero where C exceeds 1.  The first unit then already reaches the target, so K* is
max(1, K_min) up to the budget, as the oracle's; also at a target of exactly zero."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_21278_amd as enf

pytestmark = pytest.mark.gpu

# (N1, N2): one wave; several; the large box's device sort
BOXES = [(8, 8), (33, 20), (64, 64), (96, 96)]


def _spectrum(N1, N2, kind, n=3):
    rng = np.random.default_rng(N1 + 7 * N2)
    if kind == "flat":   # exactly equal energies
        return np.array([1, 1j, -1, -1j])[rng.integers(0, 4, (n, N2, N1))]
    return rng.uniform(1.0, 1.5, (n, N2, N1)) * np.exp(2j * np.pi * rng.random((n, N2, N1)))


def _plan(n, N1, N2):
    return enf.Plan(np.zeros(n + 1, dtype=np.int64), None, n_modes=(N1, N2), precision="f64", eps=1e-10, window="none")


@pytest.mark.parametrize("wide", ["0", "1"])
@pytest.mark.parametrize("k_min", [0, 1, 5])
@pytest.mark.parametrize("alphas", [(0.5, 0.0), (0.0, 0.0)])
@pytest.mark.parametrize("kind", ["spread", "flat"])   # the bucket sort and the network
@pytest.mark.parametrize("box", BOXES)
def test_negative_target(box, kind, alphas, k_min, wide, monkeypatch):
    monkeypatch.setenv("ENUFFT_EMS_WIDE", wide)
    N1, N2 = box
    f = _spectrum(N1, N2, kind)
    prm = oracle.EmsParams(k_min=k_min, alpha_min=alphas[0], alpha_max=alphas[1], w1=1.0, w2=1.0)
    ok, oks, ost = oracle.ems_batched(f, prm)
    assert (ost[:, 5] < 0.0).all() if alphas[0] > 0.0 else (ost[:, 5] == 0.0).all()
    assert (oks == max(1, k_min)).all()
    keep, ks, st = _plan(len(f), N1, N2).ems(torch.as_tensor(f, device="cuda:0"), enf.EmsParams(**prm.__dict__))
    torch.cuda.synchronize()
    assert np.array_equal(ks.cpu().numpy(), oks)
    assert np.array_equal(keep.cpu().numpy(), ok)
    assert np.allclose(st.cpu().numpy(), ost, rtol=1e-11, atol=0)


def test_negative_target_flow():
    N1, N2 = 33, 20
    f = _spectrum(N1, N2, "spread")
    fl = np.tile([6.0, 4.0, 0.02, 1e-4, 1.0, 2 * np.pi / 20000.0], (2, len(f), 1))
    fl[1, :, 4] = 0.7
    # coefficients that level the launch weights of the propagating modes
    for iy in range(N2):
        for ix in range(N1):
            w = oracle.mw_weight(ix - N1 // 2, iy - N2 // 2, fl[0, 0, 5], *fl[0, 0, :5])
            f[:, iy, ix] /= np.sqrt(w) if w > 0.0 else 1.0
    prm = oracle.EmsParams(k_min=2, alpha_min=0.5, alpha_max=0.0, w1=1.0, w2=1.0)
    ok, oks, ost = oracle.ems_flow(f, fl, prm)
    assert (ost[..., 5] < 0.0).all() and (oks == 2).all()
    keep, ks, st = _plan(len(f), N1, N2).ems_flow(torch.as_tensor(f, device="cuda:0"), fl, enf.EmsParams(**prm.__dict__))
    torch.cuda.synchronize()
    assert np.array_equal(ks.cpu().numpy(), oks)
    assert np.array_equal(keep.cpu().numpy(), ok)
    assert np.allclose(st.cpu().numpy(), ost, rtol=1e-11, atol=0)
