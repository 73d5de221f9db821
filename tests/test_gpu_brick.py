"""Small blocks advance in bricks when their launch shape is left to the
library.  The bricks evaluate a node as the marching kernel does, so states,
clocks and norm maxima must be bitwise those of the marching kernel, which a
given tile shape selects; the RMS norms are the same sums in another order
(relative difference at most the number of partial sums times 2^-53, < 1e-12
here).  Sizes at the edges of bricks, with remainders, smaller than a brick;
every kind of boundary; both precision forms; fewer stages."""
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


def _run(B, dims, metrics, q, steps, **kw):
    with B.Solver(dims, B.params_default(**kw)) as s:
        s.set_grid_metrics(metrics)
        s.set_state(q)
        s.advance(steps)
        return s.get_state(), s.clock(), s.residual_norms()


def _same(a, b):
    assert np.array_equal(a[0], b[0])
    assert a[1] == b[1] and np.array_equal(a[2][1], b[2][1])
    assert np.allclose(a[2][0], b[2][0], rtol=1e-12, atol=0)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("dims", [(8, 8, 4), (9, 9, 5), (7, 7, 3), (1, 1, 1), (3, 17, 2), (24, 20, 18), (70, 33, 41)])
def test_periodic_bricks_equal_the_march(B, prec, dims):
    print(f"[gpu-case] bricks periodic precision={prec} {dims}", flush=True)
    # a pressure jump, so that both branches of the dissipation run
    g, q = I.shock_box_case(dims, seed=5)
    _same(_run(B, dims, g.metrics, q, 3, precision=prec),
          _run(B, dims, g.metrics, q, 3, precision=prec, **TILE[prec]))


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("dims", [(4, 4, 4), (5, 5, 5), (3, 9, 13), (31, 32, 29), (32, 33, 29), (45, 37, 22)])
@pytest.mark.parametrize("bc", [(0,) * 6, (1, 2, 2, 2, 2, 2), (0, 0, 2, 2, 0, 0)])
def test_small_and_wide_bricks_equal_the_march(B, prec, dims, bc):
    """Edges and remainders of 4 x 4 x 4 bricks (up to 512 of them) and of
    8 x 8 x 4 ones, periodic and with bounded directions."""
    if any(bc) and min(dims) < 9:
        pytest.skip("a bounded direction needs its boundary layers and stencil")
    print(f"[gpu-case] bricks small and wide precision={prec} {dims} {bc}", flush=True)
    g = I.uniform_box(*dims)
    q = I.jet_state(g, 1.4, seed=sum(dims))
    kw = dict(precision=prec, bc=bc)
    _same(_run(B, dims, g.metrics, q, 2, **kw), _run(B, dims, g.metrics, q, 2, **kw, **TILE[prec]))


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("dims", [(45, 20, 37), (13, 9, 11)])
def test_curvilinear_bricks_equal_the_march(B, prec, dims):
    """Every metric component nonzero, strong noise: any multiply-add that one
    kernel contracts and the other does not shows up."""
    print(f"[gpu-case] bricks curvilinear precision={prec} {dims}", flush=True)
    g = I.wavy_grid(*dims)
    q = I.jet_state(g, 1.4, seed=9, noise=0.03)
    got = []
    for kw in ({}, TILE[prec], dict(tile_i=12, tile_j=12)):
        with B.Solver(dims, B.params_default(precision=prec, re_d=2.0e3, **kw)) as s:
            s.set_grid_coords(g.x, g.y, g.z, g.period)
            s.set_state(q)
            s.advance(4)
            got.append((s.get_state(), s.clock(), s.residual_norms()))
    _same(got[0], got[1])
    _same(got[0], got[2])


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("kind", ["domain", "cylinder", "smallest"])
def test_bounded_bricks_equal_the_march(B, prec, kind):
    print(f"[gpu-case] bricks bounded precision={prec} {kind}", flush=True)
    dims = {"domain": (26, 21, 15), "cylinder": (27, 13, 18), "smallest": (5, 5, 6)}[kind]
    g, q, bc = I.jet_cylinder_case(dims, seed=2) if kind == "cylinder" else I.jet_domain_case(dims, seed=2)
    _same(_run(B, dims, g.metrics, q, 3, precision=prec, bc=bc),
          _run(B, dims, g.metrics, q, 3, precision=prec, bc=bc, **TILE[prec]))


@pytest.mark.parametrize("prec", [0, 1])
def test_bricks_with_two_stages_and_after_a_shape_change(B, prec):
    print(f"[gpu-case] bricks two stages precision={prec}", flush=True)
    dims = (19, 11, 9)
    g, q = I.jet_box_case(dims, seed=4)
    kw = dict(precision=prec, n_stages=2, rk_alpha=(0.5, 1.0))
    a = _run(B, dims, g.metrics, q, 4, **kw)
    _same(a, _run(B, dims, g.metrics, q, 4, **kw, **TILE[prec]))
    # a solver created with a tile shape, then returned to the library's choice
    with B.Solver(dims, B.params_default(**kw, **TILE[prec])) as s:
        s.set_grid_metrics(g.metrics)
        s.set_state(q)
        s.advance(2)
        s.set_tiling(0, 0, 0)
        s.advance(2)
        _same(a, (s.get_state(), s.clock(), s.residual_norms()))


def test_failed_step_freezes_the_state(B):
    """A fixed dt far beyond stability: the flag is set by the step that
    overflows and later steps leave the state as it is."""
    print("[gpu-case] bricks failing step", flush=True)
    g, q = I.jet_box_case((12, 10, 8), seed=1)
    with B.Solver(g.dims, B.params_default(dt_fixed=1e3)) as s:
        s.set_grid_metrics(g.metrics)
        s.set_state(q)
        out = []
        for n in (20, 3):
            s.advance(n)
            x = np.empty((5, g.n))
            with pytest.raises(B.JzError):
                s.get_state(x)
            out.append(x)
        assert np.array_equal(out[0], out[1], equal_nan=True)
