"""Calls in which the workgroups of the one-launch CG give up waiting for one another: with a wait limit of 0 every
workgroup does, at the first meeting, and the call has to come to the results of the sweeps."""
import ctypes

import numpy as np
import pytest

import synth

gpu = pytest.mark.gpu
BOX = (1.0, 0.7, 0.9)


@pytest.fixture(scope="module")
def ex():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1507_05063_amd as ex

    return ex


def dev(a):
    import torch

    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def rel2(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.fixture(scope="module")
def oracle(orc):
    """The oracle's run at given iteration counts, each made once."""
    made = {}

    def run(f, g, nc, iters):
        key = (f.tobytes(), nc, tuple(iters))
        if key not in made:
            made[key] = orc.excmg(f, g, BOX, nc, 1e-10, fixed_iters=np.array(iters, dtype=np.int32), want_ext=True)
        return made[key]

    return run


def test_argument_errors():
    from paper_1507_05063_amd import _lib

    assert _lib.lib().excmg_set_wait_limit(None, 1) == _lib.ERR_ARG


# the finest grid on the chip (with and without a history to read), one-workgroup grids, and a finest grid of the
# two-step sweeps above resident ones
@gpu
@pytest.mark.parametrize("n,nc,history", [((64, 48, 32), (16, 12, 8), False), ((64, 48, 32), (16, 12, 8), True),
                                          ((128, 128, 128), (8, 8, 8), False), ((16, 16, 16), (4, 4, 4), False),
                                          ((160, 112, 144), (20, 14, 18), False)])
def test_solve(ex, oracle, n, nc, history):
    import torch

    f, g, _ = synth.sample(synth.smooth(5, BOX), n)
    s = ex.Solver(n, BOX, 1e-10, n_coarse=nc, history=history)
    want = s.solve(dev(f), dev(g))[0].clone()
    with pytest.raises(ex.ExcmgError):
        s.set_wait_limit(-1)
    s.set_wait_limit(0)
    for _ in range(2):
        u, ue, st = s.solve(dev(f), dev(g), want_ext=True)
        ref = oracle(f, g, nc, st["iters"])
        assert st["status"] == 0 and st["relres"][-1] <= 1e-10
        assert rel2(u.cpu().numpy(), ref["u"]) <= 1e-12 and rel2(ue.cpu().numpy(), ref["ut"]) <= 1e-12
        assert len(st["history"]) == (st["iters"][-1] + 1 if history else 0)
    if n != (160, 112, 144):  # there the other solver's finest grid is relaxed without the two-step sweeps
        assert torch.equal(u, ex.Solver(n, BOX, 1e-10, n_coarse=nc, two_pass_cg=True).solve(dev(f), dev(g))[0])
    s.set_wait_limit(1 << 20)
    assert torch.equal(s.solve(dev(f), dev(g))[0], want)


@gpu
@pytest.mark.parametrize("looks", [0, 1 << 20])
@pytest.mark.parametrize("n,nc", [((64, 48, 32), (16, 12, 8)), ((160, 112, 144), (20, 14, 18))])
def test_outputs_over_inputs(ex, n, nc, looks):
    """u over f or g, and the adjoint's outputs over G: a call that starts over reads its inputs again."""
    import torch

    f, g, _ = synth.sample(synth.smooth(5, BOX), n)
    s = ex.Solver(n, BOX, 1e-10, n_coarse=nc)
    s.set_wait_limit(looks)
    want = s.solve(dev(f), dev(g))[0]
    for which in (0, 1):
        fg = [dev(f), dev(g)]
        assert torch.equal(s.solve(fg[0], fg[1], u=fg[which])[0], want)
    G = dev(np.random.default_rng(0).standard_normal(want.shape))
    a, b, lam, _ = s.adjoint(G, want_lambda=True)
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    for which in range(3):
        out = [torch.empty_like(G) for _ in range(3)]
        out[which] = G.clone()
        assert ex._lib.lib().excmg_adjoint(s.handle, ptr(out[which]), *(ptr(t) for t in out), None) == 0
        assert all(torch.equal(x, y) for x, y in zip(out, (a, b, lam)))


@gpu
@pytest.mark.parametrize("graphs", [True, False])
def test_batch(ex, oracle, graphs):
    """Problems that give up beside problems that do not."""
    cases = [((64, 48, 32), (16, 12, 8)), ((64, 64, 64), (8, 8, 8)), ((16, 24, 16), (4, 6, 4)),
             ((128, 64, 96), (16, 8, 12))]
    solvers, data = [], []
    for q, (n, nc) in enumerate(cases):
        solvers.append(ex.Solver(n, BOX, 1e-10, n_coarse=nc, graphs=graphs))
        data.append(synth.sample(synth.smooth(q, BOX), n)[:2])
    for giving_up in ((1, 2), (0, 1, 2, 3), (0,), ()):
        for q, s in enumerate(solvers):
            s.set_wait_limit(0 if q in giving_up else 1 << 20)
        us, stats, _ = ex.solve_batched(solvers, [dev(f) for f, _ in data], [dev(g) for _, g in data])
        for (n, nc), (f, g), u, st in zip(cases, data, us, stats):
            ref = oracle(f, g, nc, st["iters"])
            assert rel2(u.cpu().numpy(), ref["u"]) <= 1e-12, (n, giving_up)
            assert all(r <= 1e-10 for r in st["relres"][2:])


@gpu
def test_batch_time_counts_the_sweeps(ex):
    """A problem whose finest grid gave up is done when the sweeps are, not at the give-up: its time is at least half that
    of a solver that runs the sweeps alone (the sweeps are nine tenths of it)."""
    n, nc = (64, 64, 64), (16, 16, 16)  # two direct solves, then the finest grid
    f, g, _ = synth.sample(synth.smooth(1), n)
    times = {}
    for two_pass in (True, False):
        s = ex.Solver(n, (1.0, 1.0, 1.0), 1e-10, n_coarse=nc, two_pass_cg=two_pass)
        for _ in range(3):
            s.set_wait_limit(0)
            times[two_pass] = ex.solve_batched([s], [dev(f)], [dev(g)])[2][0]
    assert times[False] >= 0.5 * times[True], times


@gpu
def test_stream_of_half_the_cus(ex):
    """A stream made for half of the CUs, where 256 workgroups cannot run together: the sweeps from the start, alone and
    in a batch that it leads, without a wait for the others."""
    import time

    import torch

    hip = ctypes.CDLL("libamdhip64.so")
    raw = ctypes.c_void_p(0)
    mask = (ctypes.c_uint32 * 8)(*[0xFFFF] * 8)
    if hip.hipExtStreamCreateWithCUMask(ctypes.byref(raw), 8, mask) != 0:
        pytest.skip("no stream with a CU mask to be had")
    n, nc = (128, 128, 128), (16, 16, 16)
    f, g, _ = (dev(v) for v in synth.sample(synth.smooth(1), n))
    part = ex.Solver(n, (1.0,) * 3, 1e-10, nc, stream=torch.cuda.ExternalStream(raw.value))
    whole = ex.Solver(n, (1.0,) * 3, 1e-10, nc)
    want = ex.Solver(n, (1.0,) * 3, 1e-10, nc, two_pass_cg=True).solve(f, g)[0]
    for s in (part, whole):
        s.set_wait_limit(1 << 22)  # a wait of more than a second
    torch.cuda.synchronize()
    t = time.perf_counter()
    u = part.solve(f, g)[0]
    us, _, _ = ex.solve_batched([part, whole], [f, f], [g, g])
    t = time.perf_counter() - t
    part.close()
    assert hip.hipStreamDestroy(raw) == 0
    assert torch.equal(u, want) and t < 0.5, t
    for v in us:
        assert torch.linalg.vector_norm(v - want) <= 1e-9 * torch.linalg.vector_norm(want)
