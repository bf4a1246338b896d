"""The in-register EMS's value sort at the edges of its forms (unit counts at and next to
the sizes where a form ends) and on the spectra that take its different routes: a
power law (buckets), repeated levels (equal values inside buckets), mostly zero
weights (the tail), and a flat spectrum under one huge peak (a crowded bucket: the
comparison network).  Same FP64 coefficients on both sides: identical selection."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_21278_amd as enf

pytestmark = pytest.mark.gpu

# (N1, N2, pairs): 63, 64 and 65 single modes, 127 .. 4,095 and 4,096 units
BOXES = [(8, 8, 0), (13, 5, 0), (16, 16, 1), (32, 17, 0), (32, 32, 0), (33, 31, 0), (64, 33, 0), (64, 48, 0),
         (64, 64, 1), (64, 64, 0)]


@pytest.mark.parametrize("wide", ["0", "1"])
@pytest.mark.parametrize("kind", ["power", "levels", "zeros", "peak"])
@pytest.mark.parametrize("box", BOXES)
def test_value_sort(box, kind, wide, monkeypatch):
    N1, N2, pairs = box
    monkeypatch.setenv("ENUFFT_EMS_WIDE", wide)
    n = 5
    rng = np.random.default_rng(N1 * 100 + N2 + pairs)
    kx = np.arange(N1) - N1 // 2
    ky = np.arange(N2) - N2 // 2
    k = np.maximum(1.0, np.hypot(kx[None, :], ky[:, None]))
    f = rng.standard_normal((n, N2, N1)) + 1j * rng.standard_normal((n, N2, N1))
    mw = None
    if kind == "power":
        f = f * 100.0 * k ** -1.5
    elif kind == "levels":    # integers: exact energies and sums
        f = rng.integers(1, 40, (n, N2, N1)) * np.array([1, 1j, -1, -1j])[rng.integers(0, 4, (n, N2, N1))]
    elif kind == "zeros":
        mw = np.where(rng.random((N2, N1)) < 0.6, 0.0, rng.uniform(0.5, 2.0, (N2, N1)))
    else:
        f = f / np.abs(f) * (1.0 + 1e-3 * rng.random((n, N2, N1)))
        f[:, N2 // 2 + 1, N1 // 2 + 1] = 1e15
    prm = oracle.EmsParams(alpha_min=0.9, alpha_max=0.9, use_pairs=pairs, exclude_dc=1)
    plan = enf.Plan(np.zeros(n + 1, dtype=np.int64), None, n_modes=(N1, N2), precision="f64", eps=1e-10, window="none")
    w = None if mw is None else torch.as_tensor(mw, device="cuda:0")
    keep, ks, st = plan.ems(torch.as_tensor(f, device="cuda:0").to(torch.complex128).contiguous(),
                            enf.EmsParams(**prm.__dict__), mode_weight=w)
    torch.cuda.synchronize()
    ok, oks, ost = oracle.ems_batched(f, prm) if mw is None else oracle.ems_batched(f, prm, mode_weight=mw)
    assert np.array_equal(ks.cpu().numpy(), oks)
    assert np.array_equal(keep.cpu().numpy(), ok)
    assert np.allclose(st.cpu().numpy(), ost, rtol=1e-11, atol=0)
