"""A batch marches its members in longer chunks after the first stage where
they leave the chunk length to the library.  Each member is still bitwise what
it is alone with the same tile shape, RMS norms included; with the library's
own tile shape too, up to the order of the RMS sums (< 1e-12).  Members joining
and leaving change the chunks of the others between steps."""
import numpy as np
import pytest

from paper_2003_09926_amd import inputs as I

pytestmark = pytest.mark.gpu

# long and short along zeta, whole and ragged chunks, one chunk only
DIMS = [(20, 14, 150), (33, 25, 64), (17, 12, 97), (16, 13, 7), (40, 30, 33)]
TILE = {0: dict(tile_i=16, tile_j=12), 1: dict(tile_i=32, tile_j=16)}


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "GPU test without a GPU"
    from paper_2003_09926_amd import binding
    binding.library()
    return binding


def _solvers(B, prec, **kw):
    out = []
    for b, d in enumerate(DIMS):
        g, q = I.jet_box_case(d, seed=20 + b)
        s = B.Solver(d, B.params_default(precision=prec, mach_j=1.2 + 0.1 * b, **kw))
        s.set_grid_metrics(g.metrics)
        s.set_state(q)
        out.append(s)
    return out


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("given", [True, False])
def test_members_of_longer_chunks(B, prec, given):
    print(f"[gpu-case] batch chunks precision={prec} tile given={given}", flush=True)
    kw = TILE[prec] if given else {}
    alone = []
    for s, n in zip(_solvers(B, prec, **kw), (3, 3, 3, 2, 2)):
        s.advance(n)
        alone.append((s.get_state(), s.clock(), s.residual_norms()))
        s.close()
    ms = _solvers(B, prec, **kw)
    with B.Batch(ms[:3]) as b:
        b.advance(1)
        b.add(ms[3])
        b.add(ms[4])
        b.advance(2)
        b.remove(ms[0])
        b.synchronize()
    for s, (q, clk, (rms, linf)) in zip(ms, alone):
        assert np.array_equal(s.get_state(), q) and s.clock() == clk
        r, l = s.residual_norms()
        assert np.array_equal(l, linf)
        assert np.array_equal(r, rms) if given else np.allclose(r, rms, rtol=1e-12, atol=0)
        s.close()
