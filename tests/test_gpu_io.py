"""States and metrics in and out: device buffers are read and written by the
kernels where they lie, anything else (host arrays, memory of another kind
passed as device memory, a buffer not aligned as doubles) goes through a copy.
All give the same bytes; a rejected state leaves the previous one; the step
size taken with a new state is the one a separate evaluation gives."""
import ctypes

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


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("dims", [(1, 1, 1), (16, 16, 1), (257, 1, 1), (37, 23, 19)])
def test_device_and_host_buffers_agree(B, prec, dims):
    import torch
    print(f"[gpu-case] buffers precision={prec} {dims}", flush=True)
    g, q = I.jet_box_case(dims, seed=6)
    got = []
    for dev in (False, True):
        with B.Solver(dims, B.params_default(precision=prec)) as s:
            m, x = (torch.from_numpy(g.metrics).cuda(), torch.from_numpy(q).cuda()) if dev else (g.metrics, q)
            s.set_grid_metrics(m)
            s.set_state(x)
            back = s.get_state(torch.empty_like(x)).cpu().numpy() if dev else s.get_state()
            assert np.array_equal(back, q)
            met = s.get_grid_metrics()
            dt = s.clock()[1]
            assert s.eval_dt()[0] == dt        # taken with the state, and evaluated on its own
            s.advance(2)
            got.append((met, dt, s.get_state(torch.empty_like(x)).cpu().numpy() if dev else s.get_state()))
    for a, b in zip(*got):
        assert np.array_equal(a, b)


def test_other_memory_goes_through_a_copy(B):
    """A pinned host buffer, and a device buffer four bytes off a double
    boundary, passed as device pointers."""
    import torch
    print("[gpu-case] pinned and misaligned buffers", flush=True)
    dims = (19, 14, 11)
    g, q = I.jet_box_case(dims, seed=7)
    lib = B.library()
    n = q.size * 8
    pinned = torch.from_numpy(q).pin_memory()
    raw = torch.zeros(n + 16, dtype=torch.uint8, device="cuda")
    raw[4:4 + n] = torch.from_numpy(q.reshape(-1).view(np.uint8)).cuda()
    torch.cuda.synchronize()
    with B.Solver(dims, B.params_default()) as s:
        s.set_grid_metrics(g.metrics)
        for ptr in (pinned.data_ptr(), raw.data_ptr() + 4):
            assert lib.jz_set_state(s._h, ctypes.c_void_p(ptr), 1) == B.JZ_OK
            assert np.array_equal(s.get_state(), q)
        raw.zero_()
        torch.cuda.synchronize()
        assert lib.jz_get_state(s._h, ctypes.c_void_p(raw.data_ptr() + 4), 1) == B.JZ_OK
        assert np.array_equal(raw[4:4 + n].cpu().numpy().view(np.float64).reshape(5, -1), q)
        assert not raw[:4].any() and not raw[4 + n:].any()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("on_device", [False, True])
def test_rejected_state_leaves_the_previous_one(B, prec, on_device):
    import torch
    print(f"[gpu-case] rejected state precision={prec} device={on_device}", flush=True)
    dims = (21, 9, 13)
    g, q = I.jet_box_case(dims, seed=8)
    put = (lambda a: torch.from_numpy(a).cuda()) if on_device else (lambda a: a)
    with B.Solver(dims, B.params_default(precision=prec)) as s:
        s.set_grid_metrics(g.metrics)
        s.set_state(put(q))
        for bad, at, code in ((np.nan, (3, -1), B.JZ_ENONFINITE), (-1.0, (0, 0), B.JZ_EINVAL), (0.0, (4, 5), B.JZ_EINVAL)):
            x = q.copy()
            x[at] = bad
            with pytest.raises(B.JzError) as ei:
                s.set_state(put(x))
            assert ei.value.code == code
            assert np.array_equal(s.get_state(), q)
        s.advance(2)
        after = s.get_state()
    with B.Solver(dims, B.params_default(precision=prec)) as s:
        s.set_grid_metrics(g.metrics)
        s.set_state(q)
        s.advance(2)
        assert np.array_equal(s.get_state(), after)


def test_many_solvers_share_the_answer_pages(B):
    """More solvers than a page of answer slots holds, from several threads;
    each reads its own clock."""
    from concurrent.futures import ThreadPoolExecutor
    import torch
    print("[gpu-case] answer slots", flush=True)
    g, q = I.jet_box_case((6, 5, 4), seed=1)

    def make(k):
        s = B.Solver(g.dims, B.params_default(dt_fixed=1e-4 * (k + 1)), stream=torch.cuda.Stream())
        s.set_grid_metrics(g.metrics)
        s.set_state(q)
        s.advance(1)
        return s

    with ThreadPoolExecutor(4) as pool:
        ss = list(pool.map(make, range(150)))
        clocks = list(pool.map(lambda s: s.clock(), ss))
    for k, (t, dt, n) in enumerate(clocks):
        assert n == 1 and t == dt == 1e-4 * (k + 1)
    for s in ss:
        s.close()


def test_answers_are_those_of_the_call(B):
    """The host watches a pinned slot for the number of its answer: solvers one
    after another in the same slot, answers of short and long queues."""
    print("[gpu-case] answers through reused slots", flush=True)
    dims = (96, 64, 40)
    g, q = I.jet_box_case(dims, seed=2)
    for steps in (1, 3, 2, 60):
        with B.Solver(dims, B.params_default()) as s:
            s.set_grid_metrics(g.metrics)
            s.set_state(q)
            t = [s.clock()[2]]
            for n in (steps, 1):
                s.advance(n)
                t.append(s.clock()[2])
            assert t == [0, steps, steps + 1]
            assert np.isfinite(s.residual_norms()[0]).all()
