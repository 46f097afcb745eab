"""A call that ends in an error leaves its outputs as they were: the data holds a NaN that only one grid of the cascade
reads, on each of its kinds (direct solves, one-launch CG, sweeps), and the handle is as before afterwards."""
import ctypes

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ex():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1507_05063_amd as ex

    return ex


def ptr(t):
    return ctypes.c_void_p(t.data_ptr())


# grids on the chip; one-workgroup grids and sweeps; direct solves alone, in one launch and in four; a finest grid that
# runs iterations in pairs
@pytest.mark.parametrize("n,nc,kw", [
    ((32, 32, 32), (4, 4, 4), {}),
    ((64, 48, 32), (16, 12, 8), {}),
    ((32, 32, 32), (4, 4, 4), {"two_pass_cg": True}),
    ((16, 16, 16), (4, 4, 4), {"two_pass_cg": True}),
    ((8, 8, 8), (8, 8, 8), {}),
    ((40, 36, 28), (20, 18, 14), {}),
    ((160, 112, 144), (20, 14, 18), {}),
])
def test_nan(ex, n, nc, kw):
    import torch

    L, s = ex._lib.lib(), ex.Solver(n, (1.0, 1.0, 1.0), 1e-10, n_coarse=nc, **kw)
    f, g, _ = (torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in synth.sample(synth.smooth(3), n))
    ext = s.levels > 1
    good = [v.clone() for v in s.solve(f, g, want_ext=ext)[:2] if v is not None] + list(s.adjoint(f)[:2])
    for l in range(s.levels):
        # a node of grid l that no coarser one has among its nodes (nor next to them in the right-hand side's stencil
        # of R, whose neighbours lie at the grid's own distance)
        step = 1 << (s.levels - 1 - l)
        bad = f.clone()
        bad[step, step, step] = float("nan")
        out = [torch.full_like(f, 7.0 + q) for q in range(3)]
        code = L.excmg_solve(s.handle, ptr(bad), ptr(g), ptr(out[0]), ptr(out[1]) if ext else None, None)
        assert code == ex._lib.ERR_NONFINITE, l
        code = L.excmg_adjoint(s.handle, ptr(bad), *(ptr(v) for v in out), None)
        assert code == ex._lib.ERR_NONFINITE, l
        for q, v in enumerate(out):
            assert bool((v == 7.0 + q).all()), (l, q)
        again = [v for v in s.solve(f, g, want_ext=ext)[:2] if v is not None] + list(s.adjoint(f)[:2])
        assert all(torch.equal(a, b) for a, b in zip(again, good)), l
