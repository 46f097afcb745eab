"""Sweep shapes of grids that run iterations in pairs alone and in two passes in a batch: a shape timed for the one form
is not used for the other.  Shapes show in the order of the partial sums only, so equal bits mean equal shapes."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

N, NC, BOX = (160, 112, 144), (20, 14, 18), (1.0, 0.7, 0.9)


@pytest.fixture(scope="module")
def ex():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1507_05063_amd as ex

    return ex


@pytest.fixture(scope="module")
def data():
    import torch

    f, g, _ = synth.sample(synth.smooth(5, BOX), N)
    return [torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in (f, g)]


@pytest.mark.parametrize("ir", [False, True])
def test_batch_after_the_tuner_of_one(ex, data, ir):
    import torch

    f, g = data
    new = lambda **kw: ex.Solver(N, BOX, 1e-10, NC, ex.FP32_IR if ir else ex.FP64, **kw)
    batch = lambda s: ex.solve_batched([s], [f], [g])[0][0].clone()
    want = batch(new())
    tuned = new()
    tuned.autotune()
    assert torch.equal(batch(tuned), want)
    # one shape set, the batch's own default: the other pass's is as it was
    some, passes = new(), new(two_pass_cg=True)
    kind = "b32" if ir else "b"
    some.set_sweep(some.levels - 1, kind, passes.get_sweep(some.levels - 1, kind))
    assert torch.equal(batch(some), want)


@pytest.mark.parametrize("ir", [False, True])
def test_single_after_the_tuner_of_batches(ex, data, ir):
    import torch

    f, g = data
    new = lambda: ex.Solver(N, BOX, 1e-10, NC, ex.FP32_IR if ir else ex.FP64)
    want, s = new().solve(f, g)[0], new()
    zc = ex.autotune_batched([s])
    assert s.get_sweep(s.levels - 1, "b32" if ir else "b")[0] == zc[0][ir]
    assert torch.equal(s.solve(f, g)[0], want)


def test_tuner_of_batches_times_what_sweeps(ex):
    """The batch's tuner times the grids that the sweeps relax, not those relaxed in one launch beside them; in a batch of
    the latter alone it times them."""
    big, small = ex.Solver(N, BOX, 1e-10, NC), ex.Solver((64, 48, 32), BOX, 1e-10, (16, 12, 8))
    zc = ex.autotune_batched([big, small])
    assert set(zc) == {0} and zc[0][0] > 0, zc
    default = ex.Solver((64, 48, 32), BOX, 1e-10, (16, 12, 8)).get_sweep(2, "a")
    assert small.get_sweep(2, "a") == default
    assert ex.autotune_batched([small])[0][0] > 0
