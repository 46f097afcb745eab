"""The direct solve of the two coarsest grids by sine transforms against the oracle's banded Cholesky, to the
repository's parity bar: a relative L2 difference of 1e-12."""
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


def dev(a):
    import torch

    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def rel2(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


# One workgroup: one unknown, 1024 unknowns, a 64-cell axis.  Four launches: one column too many for one workgroup
# (1040 unknowns), one plane, planes and columns of the largest size on each axis, ragged columns; then the larger of
# two direct grids, and both of them in three.
@pytest.mark.parametrize("n,nc", [
    ((2, 2, 2), (2, 2, 2)),
    ((17, 5, 17), (17, 5, 17)),
    ((64, 3, 9), (64, 3, 9)),
    ((3, 9, 64), (3, 9, 64)),
    ((14, 17, 6), (14, 17, 6)),
    ((64, 64, 2), (64, 64, 2)),
    ((2, 64, 64), (2, 64, 64)),
    ((8, 64, 64), (8, 64, 64)),
    ((64, 9, 31), (64, 9, 31)),
    ((26, 22, 18), (13, 11, 9)),
    ((32, 64, 48), (8, 16, 12)),
])
def test_direct_solve_matches_oracle(ex, orc, n, nc):
    box = tuple(0.04 * v for v in n)
    f, g, _ = synth.sample(synth.smooth(4, box), n)
    s = ex.Solver(n, box, 1e-11, n_coarse=nc)
    u, _, st = s.solve(dev(f), dev(g))
    u = u.cpu().numpy()
    it = np.array(st["iters"], dtype=np.int32)
    ref = orc.excmg(f, g, box, nc, 1e-11, fixed_iters=it)
    assert list(it[:2]) == [0, 0][:len(it)] and max(st["relres"][:2]) <= 1e-12
    assert rel2(u, ref["u"]) <= 1e-12
    mask = synth.boundary_mask(n)
    assert np.array_equal(u[mask], g[mask])
    dLdf, dLdg, lam, st = s.adjoint(dev(f), want_lambda=True)
    ref = orc.adjoint(f, box, nc, 1e-11, fixed_iters=np.array(st["iters"], dtype=np.int32))
    for a, k in [(lam, "lam"), (dLdf, "dLdf"), (dLdg, "dLdg")]:
        assert rel2(a.cpu().numpy(), ref[k]) <= 1e-12
    f[1, 1, 1] = np.nan
    with pytest.raises(ex.ExcmgError) as e:
        s.solve(dev(f), dev(g))
    assert e.value.code == ex._lib.ERR_NONFINITE
