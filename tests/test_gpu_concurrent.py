"""Calls from several host threads whose grids are relaxed in one launch each: such launches share the CUs, take turns
where they do not fit together, and wait for nothing else."""
import ctypes
import threading
import time

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


def case(ex, n, seed, stream):
    f, g, _ = synth.sample(synth.smooth(seed), n)
    return ex.Solver(n, (1.0, 1.0, 1.0), 1e-10, stream=stream), dev(f), dev(g)


def run(jobs):
    bad = []

    def guard(job):
        try:
            job()
        except BaseException as e:  # noqa: B902
            bad.append(e)

    ts = [threading.Thread(target=guard, args=(job,)) for job in jobs]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    if bad:
        raise bad[0]


def test_bits_of_many_threads(ex):
    """Six threads, whose launches take 4 to 256 workgroups, on streams of their own, the per-thread default stream and the
    null stream, one of them leading batches: the bits of the same calls one after another."""
    import torch

    sizes = [(16, 16, 16), (32, 32, 32), (64, 48, 32), (128, 128, 128), (96, 112, 80)]
    streams = [torch.cuda.Stream(), torch.cuda.ExternalStream(2), torch.cuda.Stream(), torch.cuda.Stream(),
               torch.cuda.default_stream()]
    own = [case(ex, n, q, s) for q, (n, s) in enumerate(zip(sizes, streams))]
    batch = [case(ex, n, q, torch.cuda.Stream()) for q, n in enumerate(sizes[1:4])]
    # (outputs made here: torch hands memory freed in one thread to another without waiting for the solvers' streams)
    out = [[torch.empty_like(f)] for _, f, _ in own] + [[torch.empty_like(f) for _, f, _ in batch]]
    torch.cuda.synchronize()

    def call(q):
        if q < len(own):
            own[q][0].solve(*own[q][1:], u=out[q][0])
        else:
            ex.solve_batched(*(list(v) for v in zip(*batch)), us=out[q])

    for q in range(len(out)):
        call(q)
    torch.cuda.synchronize()
    want = [[u.clone() for u in us] for us in out]
    torch.cuda.synchronize()

    def job(q):
        for _ in range(15):
            call(q)
            for a, b in zip(out[q], want[q]):
                assert torch.equal(a, b), q

    run([lambda q=q: job(q) for q in range(len(out))])


@pytest.mark.parametrize("per_thread", [False, True])
def test_not_behind_other_streams_work(ex, per_thread):
    """A call whose stream still has half a second of other work before it (the host's, so that no CU is taken) keeps no
    other thread's call waiting, though both need the whole chip."""
    import torch

    n = (128, 128, 128)
    hip = ctypes.CDLL("libamdhip64.so")
    pause = lambda seconds: ctypes.CFUNCTYPE(None, ctypes.c_void_p)(lambda _: time.sleep(seconds))
    short, long = pause(0.05), pause(0.5)
    slow = torch.cuda.ExternalStream(2) if per_thread else torch.cuda.Stream()
    put = lambda fn: hip.hipLaunchHostFunc(ctypes.c_void_p(slow.cuda_stream), fn, None)
    a = case(ex, n, 1, slow)
    cells, got, took, ready = torch.zeros(64, device="cuda"), [], {}, [threading.Event(), threading.Event()]
    want, out = [a[0].solve(*a[1:])[0].clone()], [torch.empty_like(a[1]), torch.empty_like(a[1])]
    torch.cuda.synchronize()

    def first():
        # a stream whose hardware queue is not this one's too
        for stream in [torch.cuda.Stream() for _ in range(16)]:
            assert put(short) == 0
            t = time.perf_counter()
            with torch.cuda.stream(stream):
                cells.add_(1.0)
            stream.synchronize()
            t = time.perf_counter() - t
            hip.hipStreamSynchronize(ctypes.c_void_p(slow.cuda_stream))
            if t < 0.02:
                got.append(stream)
                break
        ready[0].set()
        ready[1].wait(30)
        if not got:
            return
        assert put(long) == 0
        t = time.perf_counter()
        ready[0].set()
        a[0].solve(a[1], a[2], u=out[0])
        took["a"] = time.perf_counter() - t
        assert torch.equal(out[0], want[0])

    def second():
        ready[0].wait(30)
        if not got:
            ready[1].set()
            return
        b = case(ex, n, 2, got[0])
        torch.cuda.synchronize()
        want.append(b[0].solve(b[1], b[2])[0].clone())
        torch.cuda.synchronize()
        ready[0].clear()
        ready[1].set()
        ready[0].wait(30)
        time.sleep(0.1)
        t = time.perf_counter()
        b[0].solve(b[1], b[2], u=out[1])
        took["b"] = time.perf_counter() - t
        assert torch.equal(out[1], want[1])

    run([first, second])
    if not got:
        pytest.skip("no stream with another hardware queue")
    assert took["a"] > 0.3 and took["b"] < 0.1, took
