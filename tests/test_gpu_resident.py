"""The resident CG (a grid's whole FP64 relaxation in one launch, on grids that fit the chip) against the oracle, to the
repository's parity bar: a relative L2 difference of 1e-12 at the oracle's iteration counts."""
import threading

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


# One interior brick with few nodes; rows one past a brick on every axis (17, 33); bricks of every shape, ragged on
# each axis; thin grids on each axis; the largest that fits (127^3 unknowns in 256 bricks).
@pytest.mark.parametrize("n,nc,box", [
    ((8, 8, 8), (2, 2, 2), (1.0, 1.0, 1.0)),
    ((24, 8, 16), (6, 2, 4), (1.0, 0.4, 0.7)),
    ((40, 24, 16), (10, 6, 4), (1.0, 0.6, 0.5)),
    ((72, 40, 48), (18, 10, 12), (1.5, 0.8, 1.1)),
    ((96, 112, 80), (12, 14, 10), (1.0, 1.2, 0.8)),
    ((256, 8, 16), (64, 2, 4), (8.0, 0.3, 0.5)),
    ((8, 192, 24), (2, 48, 6), (0.3, 6.0, 0.8)),
    ((16, 8, 256), (4, 2, 64), (0.5, 0.25, 8.0)),
    ((160, 144, 80), (20, 18, 10), (1.0, 0.9, 0.5)),
    ((128, 128, 128), (16, 16, 16), (1.0, 1.0, 1.0)),
])
def test_grids_match_oracle(ex, orc, n, nc, box):
    p = synth.smooth(4, box)
    f, g, _ = synth.sample(p, n)
    tol = 1e-10
    s = ex.Solver(n, box, tol, n_coarse=nc, history=True)
    ug, _, st = s.solve(dev(f), dev(g))
    it = np.array(st["iters"], dtype=np.int32)
    ref = orc.excmg(f, g, box, nc, tol, fixed_iters=it)
    assert rel2(ug.cpu().numpy(), ref["u"]) <= 1e-12
    assert len(st["history"]) == it[-1] + 1 and st["history"][-1] <= tol
    free = orc.excmg(f, g, box, nc, tol)
    assert np.all(np.abs(it - free["iters"]) <= 1), (it, free["iters"])


def test_caps_zero_data_and_nan(ex, orc):
    n, nc = (32, 32, 32), (8, 8, 8)
    p = synth.smooth(1)
    f, g, _ = synth.sample(p, n)
    for cap in (1, 4):
        s = ex.Solver(n, p.box, 1e-14, n_coarse=nc, max_iters=cap)
        ug, _, st = s.solve(dev(f), dev(g), allow_noconv=True)
        assert st["status"] == ex._lib.ERR_NOCONV and st["iters"] == [0, 0, cap]
        ref = orc.excmg(f, g, p.box, nc, 1e-14, fixed_iters=np.array(st["iters"], dtype=np.int32))
        assert rel2(ug.cpu().numpy(), ref["u"]) <= 1e-12
    s = ex.Solver(n, p.box, 1e-10, n_coarse=nc)
    u, _, st = s.solve(dev(0 * f), dev(0 * g))
    assert st["iters"] == [0, 0, 0] and float(u.abs().max()) == 0.0
    f[5, 6, 7] = np.nan  # a node that only the finest grid reads
    with pytest.raises(ex.ExcmgError) as e:
        s.solve(dev(f), dev(g))
    assert e.value.code == ex._lib.ERR_NONFINITE
    f[5, 6, 7] = 0.0
    assert s.solve(dev(f), dev(g))[2]["status"] == 0  # the handle is as before


def test_threads_on_their_own_streams(ex):
    """Calls that overlap from two host threads give the bits of calls one after another."""
    import torch

    cases = [((64, 48, 32), 0), ((128, 128, 128), 3)]
    want, jobs = [], []
    for n, seed in cases:
        p = synth.smooth(seed)
        f, g, _ = synth.sample(p, n)
        stream = torch.cuda.Stream()
        s = ex.Solver(n, p.box, 1e-10, stream=stream)
        f, g = dev(f), dev(g)
        torch.cuda.synchronize()
        want.append(s.solve(f, g)[0].clone())
        jobs.append((s, f, g))
    torch.cuda.synchronize()
    bad = []

    def work(q):
        s, f, g = jobs[q]
        u = torch.empty_like(f)
        for _ in range(20):
            s.solve(f, g, u=u)
            if not torch.equal(u, want[q]):
                bad.append(q)

    ts = [threading.Thread(target=work, args=(q,)) for q in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad


def test_per_thread_default_stream(ex):
    """The per-thread default stream, which is another stream in every thread, beside a stream of its own."""
    import torch

    n, p = (64, 48, 32), synth.smooth(2)
    f, g, _ = synth.sample(p, n)
    f, g = dev(f), dev(g)
    torch.cuda.synchronize()
    want = ex.Solver(n, p.box, 1e-10).solve(f, g)[0]
    bad = []

    def work(stream):
        s = ex.Solver(n, p.box, 1e-10, stream=stream)
        u = torch.empty_like(f)
        for _ in range(20):
            s.solve(f, g, u=u)
            if not torch.equal(u, want):
                bad.append(stream)

    per_thread = torch.cuda.ExternalStream(2)  # hipStreamPerThread
    ts = [threading.Thread(target=work, args=(st,)) for st in (per_thread, per_thread, torch.cuda.Stream())]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad


# every brick kind, and strongly unequal meshsizes
@pytest.mark.parametrize("n,nc,box", [
    ((32, 32, 32), (8, 8, 8), (1.0, 1.0, 1.0)),
    ((72, 40, 48), (18, 10, 12), (1.5, 0.8, 1.1)),
    ((80, 64, 72), (20, 16, 18), (1.0, 0.8, 0.9)),
    ((96, 96, 96), (12, 12, 12), (1.0, 1.0, 1.0)),
    ((128, 96, 64), (16, 12, 8), (1.0, 0.3, 1.7)),
    ((128, 128, 128), (16, 16, 16), (1.0, 1.0, 1.0)),
])
def test_true_residual_at_a_tight_tolerance(ex, n, nc, box):
    """The stopping test sees the residual that the iteration updates; the true one is off from it by rounding, in this form
    of CG by at most about twice as much as where M p is applied anew.  A two-pass solve to 1e-15 shows how much that is
    (its true residual is that difference, and 1e-15)."""
    import torch

    f, g, _ = (dev(v) for v in synth.sample(synth.smooth(4, box), n))
    b = ex.op_rhs(f, g, n, box)

    def true(tol, **kw):
        u, _, st = ex.Solver(n, box, tol, n_coarse=nc, **kw).solve(f, g)
        for d in range(3):
            u.select(d, 0).zero_()
            u.select(d, n[2 - d]).zero_()
        return float(torch.linalg.vector_norm(b - ex.op_apply(u, n, box)) / torch.linalg.vector_norm(b)), st["iters"]

    r, it = true(1e-13)
    r2, it2 = true(1e-13, two_pass_cg=True)
    rounding = true(1e-15, two_pass_cg=True)[0]
    assert r <= 1e-13 + 2 * rounding and r2 <= 1e-13 + 2 * rounding, (r, r2, rounding)
    assert all(abs(a - c) <= 1 for a, c in zip(it, it2)), (it, it2)
