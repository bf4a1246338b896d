"""Cells split over several workgroups: the merged chunks equal the cell spread by one
workgroup, for chunk counts on both sides of the four chunks summed per round."""
import numpy as np
import pytest
import torch

import synth
from helpers import gpu_batch, make_plan, rel_l2

pytestmark = pytest.mark.gpu

# at 1,024 points a chunk: 1, 2, 4, 5, 8, 9 and 23 chunks
COUNTS = [700, 2048, 4096, 4097, 8192, 8200, 23000]


@pytest.mark.parametrize("prec,n_modes", [("f32", (64, 64)), ("f32", (16, 9)), ("f64", (33, 20)), ("f64", (64, 64))])
def test_chunks_merge_to_the_whole_cell(prec, n_modes, monkeypatch):
    b = synth.uniform_box(counts=COUNTS, n_modes=n_modes, precision=prec, window_radius=3.0, seed=11)
    b.eps = 1e-5 if prec == "f32" else 1e-10
    gb = gpu_batch(b)
    monkeypatch.setenv("ENUFFT_FWD_ITEMS_PER_SLOT", "64")
    out = {}
    for chunk in ("1024", "1000000"):
        monkeypatch.setenv("ENUFFT_FWD_CHUNK_MIN", chunk)
        plan = make_plan(gb)
        assert plan.info()["fwd_chunk_min"] == int(chunk)
        out[chunk] = [plan.type1(gb.x, gb.y, gb.h, gb.w).cpu().numpy() for _ in range(3)]
    # every chunk's grid is rounded once and every partial sum once (at most 2 x 23
    # roundings of half a unit), and the mode box holds the larger part of the spectrum
    bound = 3 * 2 * 23 * (2.0 ** -24 if prec == "f32" else 2.0 ** -53)
    for f in out["1024"]:
        for c in range(len(COUNTS)):
            assert rel_l2(f[c], out["1000000"][0][c]) <= bound, (c, rel_l2(f[c], out["1000000"][0][c]))
