"""The two-step CG sweeps (two iterations in two passes, on the grids above 2^21 unknowns) against the oracle.

Bars: whole solves at the oracle's iteration counts to a relative L2 difference of 1e-12, the repository's parity bar;
the FP32 refinement within 1% of the discretisation error; free-running counts within one of the oracle's."""
import ctypes

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

N, NC, BOX = (160, 112, 144), (20, 14, 18), (1.0, 0.7, 0.9)  # 159 x 111 x 143: ragged tiles on every axis


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
def data():
    p = synth.smooth(5, BOX)
    return synth.sample(p, N)


@pytest.fixture(scope="module")
def oracle(orc, data):
    """The oracle's run for a tolerance and iteration counts (None: its own), each made once."""
    made = {}

    def run(tol, iters=None):
        key = (tol, None if iters is None else tuple(int(v) for v in iters))
        if key not in made:
            made[key] = orc.excmg(data[0], data[1], BOX, NC, tol, fixed_iters=iters)
        return made[key]

    return run


# every tile height; chunks of 2 planes (a chunk shorter than the sweep's lag), one that leaves a short last chunk, and
# the whole column
@pytest.mark.parametrize("ty", [4, 8, 16])
@pytest.mark.parametrize("zc,nt", [(2, 0), (10, 1), (144, 0)])
def test_shapes_match_oracle(ex, oracle, data, ty, zc, nt):
    f, g, _ = data
    tol = 1e-10
    s = ex.Solver(N, BOX, tol, n_coarse=NC, history=True)
    for kind in ("a", "b", "a_first", "b_first"):
        s.set_sweep(s.levels - 1, kind, (zc, 2, nt, ty))
    ug, _, st = s.solve(dev(f), dev(g))
    it = np.array(st["iters"], dtype=np.int32)
    ref = oracle(tol, it)
    assert rel2(ug.cpu().numpy(), ref["u"]) <= 1e-12
    assert len(st["history"]) == it[-1] + 1 and st["history"][-1] <= tol < st["history"][-2]
    free = oracle(tol)
    assert np.all(np.abs(it - free["iters"]) <= 1), (it, free["iters"])


# iteration caps: a pair that makes one iteration only (odd caps), and a solve that ends inside the first pair
@pytest.mark.parametrize("cap", [1, 2, 3, 6])
def test_iteration_caps(ex, oracle, data, cap):
    f, g, _ = data
    s = ex.Solver(N, BOX, 1e-14, n_coarse=NC, max_iters=cap)
    ug, _, st = s.solve(dev(f), dev(g), allow_noconv=True)
    it = np.array(st["iters"], dtype=np.int32)
    assert list(it) == [0, 0, cap, cap]
    ref = oracle(1e-14, it)
    assert rel2(ug.cpu().numpy(), ref["u"]) <= 1e-12


@pytest.mark.parametrize("ty,depth", [(4, 2), (8, 2), (16, 2), (16, 3)])
def test_fp32_shapes(ex, oracle, data, ty, depth):
    f, g, u = data
    tol = 1e-13
    s = ex.Solver(N, BOX, tol, n_coarse=NC, precision=ex.FP32_IR)
    for kind in ("a32", "b32"):
        s.set_sweep(s.levels - 1, kind, (10, depth, 1, ty))
    ug, _, st = s.solve(dev(f), dev(g))
    assert st["ir_outer"][-1] >= 1
    ref = oracle(tol)
    rms = lambda a: float(np.sqrt(np.mean(np.square(a))))
    assert rms(ug.cpu().numpy() - ref["u"]) <= 0.01 * rms(ref["u"] - u)


def test_outputs_may_alias_inputs(ex, data):
    """The sweeps keep a vector in an output array: an output that is also an input gives the same values (the solve's
    u over f or g, the adjoint's dL/dg over G), and so does an output aligned to 8 bytes only."""
    import torch

    f, g, _ = data
    s = ex.Solver(N, BOX, 1e-10, n_coarse=NC)
    want = s.solve(dev(f), dev(g))[0]
    for which in (0, 1):
        fg = [dev(f), dev(g)]
        assert torch.equal(s.solve(fg[0], fg[1], u=fg[which])[0], want)
    odd = torch.empty(want.numel() + 1, dtype=torch.float64, device="cuda")[1:].view(want.shape)
    assert torch.equal(s.solve(dev(f), dev(g), u=odd)[0], want)
    G = dev(np.random.default_rng(0).standard_normal(want.shape))
    a, b, _, _ = s.adjoint(G)
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    df = torch.empty_like(G)
    assert ex._lib.lib().excmg_adjoint(s.handle, ptr(G), ptr(df), ptr(G), None, None) == 0  # dL/dg over G
    assert torch.equal(df, a) and torch.equal(G, b)


def test_thin_grid(ex):
    """One tile row, narrower than the tile on y, by the finest grid's true residual (no oracle at this shape): the
    stopping test's recursive residual and the true one differ by rounding, far below tol at 1e-10."""
    import torch

    n, box = (2048, 16, 128), (16.0, 0.125, 1.0)
    p = synth.smooth(2, box)
    f, g, _ = (dev(v) for v in synth.sample(p, n))
    s = ex.Solver(n, box, 1e-10)
    u, _, st = s.solve(f, g)
    b = ex.op_rhs(f, g, n, box)
    z = u.clone()
    for d in range(3):
        z.select(d, 0).zero_()
        z.select(d, n[2 - d]).zero_()
    r = torch.linalg.vector_norm(b - ex.op_apply(z, n, box)) / torch.linalg.vector_norm(b)
    assert float(r) <= 1.01e-10
