"""The anisotropic exponent tv_alpha: 1/2 and any other value run in separate
instantiations of the stage kernels, so a batch that mixes them, or that a
member with another exponent joins after its step was captured, must still
give every member bitwise what it computes alone."""
import numpy as np
import pytest

from paper_2003_09926_amd import inputs as I

pytestmark = pytest.mark.gpu

DIMS = [(24, 20, 18), (17, 13, 11), (33, 12, 9)]
ALPHA = [0.5, 0.5, 0.7]
TILE = {0: (16, 12), 1: (32, 16)}


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "GPU test without a GPU"
    from paper_2003_09926_amd import binding
    binding.library()
    return binding


def _solver(B, prec, dims, alpha):
    g, q = I.jet_box_case(dims, seed=3)
    s = B.Solver(dims, B.params_default(precision=prec, tv_alpha=alpha, tile_i=TILE[prec][0], tile_j=TILE[prec][1]))
    s.set_grid_metrics(g.metrics)
    s.set_state(q)
    return s


@pytest.mark.parametrize("prec", [0, 1])
def test_batch_of_mixed_exponents(B, prec):
    print(f"[gpu-case] mixed exponents precision={prec}", flush=True)
    alone = []
    for d, a, n in zip(DIMS, ALPHA, (4, 4, 2)):
        with _solver(B, prec, d, a) as s:
            s.advance(n)
            alone.append((s.get_state(), s.residual_norms(), s.clock()))
    # the general exponent changes the result, so the mix is no idle test
    with _solver(B, prec, DIMS[2], 0.5) as s:
        s.advance(2)
        assert not np.array_equal(s.get_state(), alone[2][0])
    ms = [_solver(B, prec, d, a) for d, a in zip(DIMS, ALPHA)]
    with B.Batch(ms[:2]) as b:
        b.advance(2)          # captured with the square-root kernels
        b.add(ms[2])
        b.advance(2)
        b.synchronize()
    for s, (q, (rms, linf), clk) in zip(ms, alone):
        assert np.array_equal(s.get_state(), q)
        r2, l2 = s.residual_norms()
        assert np.array_equal(r2, rms) and np.array_equal(l2, linf) and s.clock() == clk
        s.close()
