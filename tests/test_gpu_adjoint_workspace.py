"""Workspace of the banded adjoint and of the reconstruction: the column spectra are held
for a group of cells at a time, the groups shrink with the room ENUFFT_ALLOC_CAP_MB leaves
(down to one cell) instead of refusing the call, and one buffer serves both.  Results do
not depend on the grouping.  A first call may also stand inside a stream capture."""
import numpy as np
import pytest
import torch

import synth
from helpers import gpu_batch, make_plan

pytestmark = pytest.mark.gpu

N = 11
PER_CELL = 2 * 128 * 33 * 2 * 8   # two sets of 128 x 33 complex FP64 columns (64 x 64 modes, sigma 2)


def _batch(prec="f64"):
    b = synth.uniform_box(counts=[40 + 700 * (c % 3) for c in range(N)], n_modes=(64, 64), precision=prec,
                          window_radius=3.0, seed=5)
    b.eps = 1e-10 if prec == "f64" else 1e-6
    return b


def _calls(gb, plan):
    rng = np.random.default_rng(8)
    g = torch.as_tensor(rng.standard_normal((N, 64, 64)) + 1j * rng.standard_normal((N, 64, 64)),
                        device="cuda:0").to(plan.cdtype)
    keep = torch.as_tensor(rng.integers(0, 2, (N, 64, 64)), device="cuda:0", dtype=torch.uint8)
    adj = lambda: list(plan.adjoint(gb.x, gb.y, gb.h, gb.w, g))
    rec = lambda: list(plan.reconstruct(gb.x, gb.y, gb.h, gb.w, g, keep))
    return adj, rec


def _run(gb, plan, first="adj"):
    adj, rec = _calls(gb, plan)
    a, r = (adj(), rec()) if first == "adj" else (rec(), adj())
    torch.cuda.synchronize()
    return (a + r) if first == "adj" else (r + a)


def _same(u, v):
    return all(torch.equal(p, q) for p, q in zip(u, v) if p is not None)


@pytest.mark.parametrize("first", ["adj", "rec"])
@pytest.mark.parametrize("cells", [0, 1, 3, N - 1, N])
def test_groups_shrink_with_the_room(cells, first, monkeypatch):
    gb = gpu_batch(_batch())
    ref = _run(gb, make_plan(gb))
    plan = make_plan(gb)
    before = plan.info()["workspace_bytes"]
    # room for that many cells' spectra and half a cell's more (the item lists are small)
    monkeypatch.setenv("ENUFFT_ALLOC_CAP_MB", repr((before + (cells + 0.5) * PER_CELL) / 2.0 ** 20))
    got = _run(gb, plan, first)
    grown = plan.info()["workspace_bytes"] - before
    held = max(1, cells)
    assert held * PER_CELL <= grown < (held + 0.5) * PER_CELL   # one buffer, of that many cells
    assert _same(got, ref)


def test_chunks_under_a_cap(monkeypatch):
    """A capped FP64 plan splits its cells as before the finer chunks, whose grids take room."""
    b = synth.uniform_box(counts=[40000, 300], n_modes=(32, 32), precision="f64", window_radius=3.0, seed=5)
    b.eps = 1e-10
    gb = gpu_batch(b)
    fine = make_plan(gb).info()
    monkeypatch.setenv("ENUFFT_FWD_CHUNK_MIN", "16384")
    coarse = make_plan(gb).info()
    monkeypatch.delenv("ENUFFT_FWD_CHUNK_MIN")
    monkeypatch.setenv("ENUFFT_ALLOC_CAP_MB", repr((coarse["workspace_bytes"] + 64) / 2.0 ** 20))
    capped = make_plan(gb).info()
    assert fine["n_items_fwd"] > coarse["n_items_fwd"] == capped["n_items_fwd"]
    assert fine["workspace_bytes"] > coarse["workspace_bytes"] == capped["workspace_bytes"]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("warm", ["adj", "rec", None])
def test_first_call_inside_a_capture(prec, warm):
    gb = gpu_batch(_batch(prec))
    ref = _run(gb, make_plan(gb))
    plan = make_plan(gb)
    adj, rec = _calls(gb, plan)
    if warm:
        adj() if warm == "adj" else rec()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = (adj() if warm != "adj" else []) + (rec() if warm != "rec" else [])
    want = (ref[:3] if warm != "adj" else []) + (ref[3:] if warm != "rec" else [])
    for _ in range(3):
        for t in out:
            if t is not None:
                t.fill_(-1)
        graph.replay()
        torch.cuda.synchronize()
        assert _same(out, want)
        assert _same(_run(gb, plan), ref)   # eager calls between the replays
