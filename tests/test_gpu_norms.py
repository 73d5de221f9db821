"""The norms a step leaves (reduced over the columns of each tile, then over the
tiles) against those of the residual field itself, for tiles of whole and
partial waves, one tile and many, bricks and the library's own shape.  FP64:
the same values summed in another order (2^-53 times the number of nodes, <
1e-11); FP32-flux: the residual of the first stage and of the residual launch
may differ by float roundings of their terms (2^-24 times some tens of terms,
< 1e-5 of the largest)."""
import numpy as np
import pytest

from paper_2003_09926_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "GPU test without a GPU"
    from paper_2003_09926_amd import binding
    binding.library()
    return binding


@pytest.mark.parametrize("dims", [(40, 30, 22), (11, 5, 3)])
@pytest.mark.parametrize("prec,tile,kchunk", [(0, (0, 0), 0), (0, (16, 12), 0), (0, (16, 16), 5), (0, (32, 8), 0),
                                              (0, (12, 12), 3), (0, (28, 12), 0), (1, (0, 0), 0), (1, (32, 16), 0),
                                              (1, (12, 12), 4), (1, (28, 20), 0)])
def test_norms_are_those_of_the_residual(B, prec, tile, kchunk, dims):
    print(f"[gpu-case] norms precision={prec} tile={tile} kchunk={kchunk} {dims}", flush=True)
    g = I.wavy_grid(*dims)
    q = I.jet_state(g, 1.4, seed=2, noise=0.03)
    with B.Solver(dims, B.params_default(precision=prec, tile_i=tile[0], tile_j=tile[1], kchunk=kchunk,
                                         re_d=2.0e3)) as s:
        s.set_grid_coords(g.x, g.y, g.z, g.period)
        s.set_state(q)
        r = np.asarray(s.eval_residual()).reshape(5, -1)
        s.advance(1)
        rms, linf = s.residual_norms()
    tol = dict(rtol=1e-5, atol=1e-5 * np.abs(r).max()) if prec else dict(rtol=1e-11, atol=0)
    assert np.allclose(rms, np.sqrt((r * r).mean(axis=1)), **tol)
    assert np.allclose(linf, np.abs(r).max(axis=1), **tol)
