"""A block by itself whose launch shape is left to the library marches in chunks
chosen for it alone: down to one or two planes where its tiles leave CUs idle.
Chunks only split the work: states, clocks and norm maxima must be bitwise
those of a given tile shape with its longer chunks, the RMS norms the same sums
in another order (relative difference at most the number of partial sums times
2^-53, < 1e-12 here).  Blocks with fewer of the finest tiles than chunks, ragged
last chunks, long thin blocks; every kind of boundary; both precision forms."""
import numpy as np
import pytest

from paper_2003_09926_amd import inputs as I

pytestmark = pytest.mark.gpu

TILE = {0: dict(tile_i=16, tile_j=12), 1: dict(tile_i=32, tile_j=16)}


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "GPU test without a GPU"
    from paper_2003_09926_amd import binding
    binding.library()
    return binding


def _advance(B, g, q, steps, bc, **kw):
    with B.Solver(g.dims, B.params_default(bc=bc, **kw)) as s:
        s.set_grid_metrics(g.metrics)
        s.set_state(q)
        s.advance(steps)
        return s.get_state(), s.clock(), s.residual_norms()


def _same(a, b):
    assert np.array_equal(a[0], b[0])
    assert a[1] == b[1] and np.array_equal(a[2][1], b[2][1])
    assert np.allclose(a[2][0], b[2][0], rtol=1e-12, atol=0)


@pytest.mark.parametrize("prec,dims,steps", [
    (0, (48, 48, 32), 2), (0, (64, 48, 47), 2),
    (0, (1, 1, 1100), 1),   # (node noise on so fine a line overflows in a second step, in any shape)
    (0, (130, 120, 6), 2), (0, (33, 140, 37), 2), (1, (96, 64, 96), 2), (1, (33, 200, 67), 2), (1, (200, 130, 9), 2)])
def test_own_chunks_equal_given_tiles(B, prec, dims, steps):
    print(f"[gpu-case] own chunks precision={prec} {dims}", flush=True)
    g, q = I.jet_box_case(dims, seed=sum(dims))
    a = _advance(B, g, q, steps, (0,) * 6, precision=prec)
    _same(a, _advance(B, g, q, steps, (0,) * 6, precision=prec, **TILE[prec]))


@pytest.mark.parametrize("prec,dims", [(0, (70, 52, 49)), (1, (101, 70, 83))])
def test_own_chunks_of_a_bounded_block(B, prec, dims):
    print(f"[gpu-case] own chunks bounded precision={prec} {dims}", flush=True)
    g = I.uniform_box(*dims)
    q = I.jet_state(g, 1.4, seed=3)
    bc = (1, 2, 2, 2, 2, 2)
    a = _advance(B, g, q, 2, bc, precision=prec)
    _same(a, _advance(B, g, q, 2, bc, precision=prec, **TILE[prec]))


def test_a_tight_workspace_and_a_shape_change(B, monkeypatch):
    """A workspace that holds the finest tiles only (the longer chunks fit
    it), and a solver returned from a given shape to the library's choice."""
    print("[gpu-case] own chunks, tight workspace", flush=True)
    dims = (48, 48, 32)
    g, q = I.jet_box_case(dims, seed=7)
    want = _advance(B, g, q, 2, (0,) * 6)
    with B.Solver(dims, B.params_default(**TILE[0])) as s:
        s.set_grid_metrics(g.metrics)
        s.set_state(q)
        s.advance(1)
        s.set_tiling(0, 0, 0)
        s.advance(1)
        _same(want, (s.get_state(), s.clock(), s.residual_norms()))
    tight = B.workspace_bytes(dims, B.params_default(**TILE[0]))
    assert tight < B.workspace_bytes(dims, B.params_default())
    monkeypatch.setattr(B, "workspace_bytes", lambda *a: tight)
    _same(want, _advance(B, g, q, 2, (0,) * 6))
