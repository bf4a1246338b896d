"""The chunk size that FP64 plans choose for themselves: cells stay whole where the split
would cost more than the idle workgroups, and split where few cells leave the chip idle;
the coefficients are those of the plain 16,384-point chunks to rounding."""
import numpy as np
import pytest
import torch

import synth
from helpers import gpu_batch, make_plan, rel_l2

pytestmark = pytest.mark.gpu


# cells, points, modes, eps, items at least and at most
@pytest.mark.parametrize("cells,points,n,eps,lo,hi", [
    (300, 3000, 16, 1e-4, 300, 300),      # two rounds of short items: whole
    (300, 3000, 32, 1e-8, 300, 300),
    (200, 6000, 64, 1e-10, 200, 200),     # one round: whole
    (1, 2000, 64, 1e-4, 1, 2),            # a transform's cost against few points
    (1, 2000, 32, 1e-10, 2, 4),
    (1, 60000, 64, 1e-8, 8, 24),          # the last chunk's sum bounds the split
    (40, 8000, 64, 1e-8, 80, 160),
    (600, 300, 64, 1e-8, 600, 600),       # more than two cells per workgroup: left alone
])
def test_chunks(cells, points, n, eps, lo, hi, monkeypatch):
    b = synth.uniform_box(counts=[points] * cells, n_modes=(n, n), precision="f64", window_radius=3.0, seed=13)
    b.eps = eps
    gb = gpu_batch(b)
    plan = make_plan(gb)
    i = plan.info()
    f = plan.type1(gb.x, gb.y, gb.h, gb.w).cpu().numpy()
    print(cells, points, n, eps, "items", i["n_items_fwd"], "chunk", i["fwd_chunk_min"], flush=True)
    assert lo <= i["n_items_fwd"] <= hi
    # the reported size is that of the schedule
    assert i["fwd_chunk_min"] <= 16384
    assert i["n_items_fwd"] == cells * max(1, -(-points // i["fwd_chunk_min"]))
    monkeypatch.setenv("ENUFFT_FWD_CHUNK_MIN", "16384")
    plan = make_plan(gb)
    assert plan.info()["fwd_chunk_min"] == 16384
    g = plan.type1(gb.x, gb.y, gb.h, gb.w).cpu().numpy()
    # both round every partial sum once (at most 24 chunks), and LDS sums in any order
    for c in range(0, cells, max(1, cells // 4)):
        assert rel_l2(f[c], g[c]) <= 24 * 64 * 2.0 ** -53
