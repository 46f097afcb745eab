"""Batches of different sizes led by one solver on one workspace, whose rounds have the same launches: every call reads
its own lists (a cached graph of the other call's would read them at that call's places)."""
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


# (n of the batch's problems, those of the larger batch alone): the resident CG's launches, and with two_pass the
# sweeps'.  The additional problems have two grids, so the third and later rounds of both batches launch the same.
@pytest.mark.parametrize("two_pass,n,count,more", [(False, (16, 16, 16), 4, 1), (False, (16, 24, 16), 1, 1),
                                                   (True, (32, 32, 32), 2, 1), (True, (32, 32, 32), 1, 6)])
@pytest.mark.parametrize("larger_first", [True, False])
def test_counts_in_turn(ex, orc, two_pass, n, count, more, larger_first):
    import torch

    nc = tuple(v // 4 for v in n)
    cases = [(n, nc)] * count + [((8, 8, 8), (4, 4, 4))] * more
    solvers, data = [], []
    for q, (m, c) in enumerate(cases):
        p = synth.smooth(q, (1.0, 0.8, 1.1))
        data.append(synth.sample(p, m)[:2])
        solvers.append(ex.Solver(m, p.box, 1e-10, n_coarse=c, two_pass_cg=two_pass))
    ws = torch.zeros(ex.batch_workspace_bytes(len(cases)), dtype=torch.uint8, device="cuda")
    for call in range(4):
        k = len(cases) if larger_first == (call % 2 == 0) else count
        # other data in every call
        scale = 1.0 + call
        fg = [(scale * f, scale * g) for f, g in data[:k]]
        dev = [[torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in pair] for pair in fg]
        us, stats, _ = ex.solve_batched(solvers[:k], [d[0] for d in dev], [d[1] for d in dev], workspace=ws)
        for (f, g), (m, c), u, st in zip(fg, cases, us, stats):
            ref = orc.excmg(f, g, (1.0, 0.8, 1.1), c, 1e-10, fixed_iters=np.array(st["iters"], dtype=np.int32))
            assert np.linalg.norm(u.cpu().numpy() - ref["u"]) <= 1e-12 * np.linalg.norm(ref["u"]), (call, m)
    if count + more > 1:
        replays, captures = solvers[0].batch_graph_counts()
        assert replays > 0 and captures > 0
