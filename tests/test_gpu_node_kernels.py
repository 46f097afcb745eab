"""The right-hand side and the transposes of the adjoint at the edges of their tiles (64 x 4 nodes, columns of 8 planes),
against the oracle at the tolerances of the other tests of the two: 1e-13 and 1e-12 of the largest entry."""
import numpy as np
import pytest

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


def relmax(a, b):
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


SIZES = [(2, 2, 2), (3, 3, 7), (62, 3, 6), (63, 4, 8), (64, 7, 9), (2, 8, 15), (64, 2, 16)]


@pytest.mark.parametrize("n", SIZES + [(65, 5, 17), (127, 9, 10), (130, 2, 33)])
def test_rhs(ex, orc, n):
    rng = np.random.default_rng(7)
    f, g = (rng.standard_normal((n[2] + 1, n[1] + 1, n[0] + 1)) for _ in range(2))
    box = (1.0, 0.7, 1.3)
    b = ex.op_rhs(dev(f), dev(g), n, box).cpu().numpy()
    assert relmax(b, orc.rhs(f, g, box)) <= 1e-13


@pytest.mark.parametrize("n", SIZES)
def test_adjoint(ex, orc, n):
    """A single grid, solved directly; dLdf is overwritten whatever it held, and so is dLdg."""
    rng = np.random.default_rng(8)
    G = rng.standard_normal((n[2] + 1, n[1] + 1, n[0] + 1))
    box = tuple(0.1 * v for v in n)
    dLdf, dLdg, lam, _ = ex.Solver(n, box, 1e-10, n_coarse=n).adjoint(dev(G), want_lambda=True)
    ref = orc.adjoint(G, box, n, 1e-10)
    for a, k in [(lam, "lam"), (dLdf, "dLdf"), (dLdg, "dLdg")]:
        assert relmax(a.cpu().numpy(), ref[k]) <= 1e-12


# one axis as long as a call may have it, on each axis (the other two as short as they come)
@pytest.mark.parametrize("n", [(70000, 2, 3), (3, 65000, 2), (2, 3, 65000)])
def test_rhs_long_axis(ex, orc, n):
    test_rhs(ex, orc, n)


def test_rhs_time_of_a_thin_grid(ex):
    """Launches follow the faces, not the longest axis squared: as many nodes in a thin box take less than ten times the
    time of a cube (with the latter, 50 times)."""
    import time

    import torch

    took = []
    for n in ((64, 64, 64), (16384, 4, 4)):
        f = torch.ones((n[2] + 1, n[1] + 1, n[0] + 1), dtype=torch.float64, device="cuda")
        times = []
        for _ in range(20):
            t = time.perf_counter()
            ex.op_rhs(f, f, n, (1.0, 1.0, 1.0))
            times.append(time.perf_counter() - t)
        took.append(sorted(times)[10])
    assert took[1] < 10 * took[0], took
