"""Batches whose grids are solved in one launch each (the direct solves and the resident CG), against the oracle to the
repository's parity bar: a relative L2 difference of 1e-12 at the batch's iteration counts."""
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


# (n, coarsest): direct grids of one unknown, of 1024, above it, and in two sizes together; resident grids of one brick,
# ragged on each axis, thin, of unlike brick kinds, and together more than one launch takes
BATCHES = {
    "direct": [((2, 2, 2), (2, 2, 2)), ((17, 17, 5), (17, 17, 5)), ((14, 17, 6), (14, 17, 6)),
               ((8, 64, 64), (8, 64, 64)), ((26, 22, 18), (13, 11, 9))],
    "one brick": [((8, 8, 8), (2, 2, 2))],
    "ragged": [((72, 40, 48), (18, 10, 12)), ((24, 8, 16), (6, 2, 4)), ((256, 8, 16), (64, 2, 4)),
               ((16, 8, 256), (4, 2, 64)), ((8, 192, 24), (2, 48, 6)), ((40, 24, 16), (10, 6, 4))],
    "many": [((64, 64, 64), (16, 16, 16))] * 5 + [((128, 128, 64), (16, 16, 8)), ((32, 32, 32), (4, 4, 4)),
                                                  ((96, 112, 80), (12, 14, 10))],
}


@pytest.mark.parametrize("name", BATCHES)
@pytest.mark.parametrize("graphs", [True, False])
def test_batch_matches_oracle(ex, orc, name, graphs):
    cases, solvers, fs, gs = BATCHES[name], [], [], []
    for q, (n, nc) in enumerate(cases):
        box = tuple(0.02 * v for v in n)
        f, g, _ = synth.sample(synth.smooth(q, box), n)
        solvers.append(ex.Solver(n, box, 1e-10, n_coarse=nc, graphs=graphs))
        fs.append(f)
        gs.append(g)
    for _ in range(2):
        us, stats, ms = ex.solve_batched(solvers, [dev(f) for f in fs], [dev(g) for g in gs])
    for (n, nc), f, g, u, st, t in zip(cases, fs, gs, us, stats, ms):
        box = tuple(0.02 * v for v in n)
        ref = orc.excmg(f, g, box, nc, 1e-10, fixed_iters=np.array(st["iters"], dtype=np.int32))
        u = u.cpu().numpy()
        assert np.linalg.norm(u - ref["u"]) <= 1e-12 * np.linalg.norm(ref["u"]), n
        assert np.array_equal(u[synth.boundary_mask(n)], g[synth.boundary_mask(n)])
        assert all(r <= 1e-10 for r in st["relres"][:st["levels"]]) and t > 0.0
