"""What the speed of this framework is measured on: solves, differentiated solves, batches and single steps.

A case is a dict of plain values.  `kind` says which public entry points a pass goes through:
  solve     Solver.solve (u, and with `ext` the sixth-order u~), then with `grad` Solver.gradient
  autograd  autograd.solve and the gradients of a loss with respect to f and g (the adjoint solve)
  batch     solve_batched over `count` problems of uneven sizes
  steps     op_rhs, op_apply, op_exp_finite and op_exp_true on one grid
Inputs are seeded smooth fields u = sum_k a_k sin sin sin + exp(.)/10 (the fields of the benchmark), evaluated on the
GPU; f is the field's Laplacian, g the field on the boundary.
"""
import math
import random

import numpy as np
import torch

import paper_1507_05063_amd as ex
from paper_1507_05063_amd import autograd

F64 = torch.float64


def _solve(name, n, coarse=(0, 0, 0), box=(1.0, 1.0, 1.0), tol=1e-10, mixed=False, ext=True, grad=True, tuned=False,
           kind="solve"):
    c = dict(kind=kind, nx=n[0], ny=n[1], nz=n[2], cx=coarse[0], cy=coarse[1], cz=coarse[2], lx=box[0], ly=box[1],
             lz=box[2], tol=tol, mixed=mixed, ext=ext, grad=grad, tuned=tuned)
    return dict(c, name=name) if name else c


def _batch(name, count, small, mixed, sizes):
    c = dict(kind="batch", count=count, small=small, mixed=mixed, tol=1e-10, sizes=sizes)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call in use: a coupling loop or a test calls it again and again; launches and round trips count
        _solve("solve 32", (32, 32, 32)),
        # a small anisotropic box with counts that are no powers of two
        _solve("solve 96x48x80", (96, 48, 80), box=(1.5, 0.8, 1.1)),
        # the five-grid workload doubled once: an ordinary call, still bound by latency as much as by bytes
        _solve("solve 128", (128, 128, 128)),
        # counts that halve only a few times, so that the two direct solves are large (26x22x18 and 52x44x36)
        _solve("solve 208x176x144", (208, 176, 144), box=(1.3, 1.1, 0.9)),
        # a tight tolerance, as for errors at the discretisation limit: many CG iterations on the finest grids
        _solve("solve 256 tight", (256, 256, 256), tol=1e-13, grad=False),
        # large and uneven, used as the README does, without the autotuner
        _solve("solve 320x448x256", (320, 448, 256), coarse=(10, 14, 8), box=(1.0, 1.4, 0.8)),
        # the benchmark's workload: 512^3, autotuned once, u, u~ and the gradient
        _solve("solve 512 tuned", (512, 512, 512), tuned=True),
        # unequal meshsizes, FP32 sweeps inside FP64 refinement: the largest grid
        _solve("mixed 1024x512x256", (1024, 512, 256), coarse=(8, 4, 2), mixed=True, ext=False, grad=False),
        # the differentiation workload: forward and adjoint solve
        _solve("autograd 256", (256, 256, 256), ext=False, grad=False, kind="autograd"),
        # a third of the batched workload: uneven sizes and aspect ratios, FP32 refinement
        _batch("batch 32 mixed", 32, False, True, 4),
        # many small problems at once in FP64
        _batch("batch 24 small", 24, True, False, 7),
        # the single steps on one grid, as a program of its own solver calls them
        _solve("steps 192x128x160", (192, 128, 160), box=(1.2, 0.8, 1.0), kind="steps"),
    ]


def draw(rng):
    """One more case of the ranges that the listed ones cover."""
    kind = rng.choices(["solve", "autograd", "batch", "steps"], [12, 2, 2, 2])[0]
    if kind == "batch":
        return _batch(None, rng.randint(4, 32), rng.random() < 0.5, rng.random() < 0.5, rng.randrange(1 << 20))
    # 32^3 to 2^27 nodes (less where a pass costs more), edges within a factor of about three of one another
    most = {"solve": 1.3e8, "autograd": 8e6, "steps": 1.6e7}[kind]
    u = math.exp(rng.uniform(math.log(3.3e4), math.log(most)))
    shape = [rng.uniform(0.6, 1.7) for _ in range(3)]
    k = (u / (shape[0] * shape[1] * shape[2])) ** (1 / 3)
    target = [k * v for v in shape]
    top = rng.choice([6, 10, 16, 28])  # cells on the longest axis of the coarsest grid, about
    levels = max(3, 1 + round(math.log2(max(target) / top)))
    coarse = [max(2, 2 * round(t / 2 ** levels)) for t in target]
    if max(coarse) < 4:
        coarse[rng.randrange(3)] = 4
    n = [c << (levels - 1) for c in coarse]
    while n[0] * n[1] * n[2] > 1.36e8:
        n[n.index(max(n))] //= 2
        coarse = [v >> (levels - 1) for v in n]
        if min(coarse) < 2 or any(c % 2 for c in coarse):
            n = [c * 2 ** (levels - 1) for c in (4, 4, 4)]
            coarse = [4, 4, 4]
    # meshsizes within a factor of about 1.5 of one another
    m = max(n)
    box = [round(v / m * rng.uniform(0.8, 1.25), 3) for v in n]
    mixed = kind == "solve" and rng.random() < 0.3
    small = n[0] * n[1] * n[2] < 4e6
    tol = rng.choice([1e-9, 1e-10, 1e-11, 1e-13]) if n[0] * n[1] * n[2] < 2e7 and kind == "solve" else 1e-10
    explicit = rng.random() < 0.7
    return _solve(None, n, tuple(coarse) if explicit else (0, 0, 0), tuple(box), tol, mixed, rng.random() < 0.6,
                  rng.random() < 0.6, kind == "solve" and small and rng.random() < 0.2, kind)


# ------------------------------------------------------------------------------------------------------- inputs


def _axes(n, box):
    """Node coordinates over the box edge, per axis, shaped to broadcast to (z, y, x)."""
    shapes = ((1, 1, -1), (1, -1, 1), (-1, 1, 1))
    return [(torch.arange(n[d] + 1, dtype=F64, device="cuda") / n[d]).reshape(shapes[d]) for d in range(3)]


def _field(n, box, seed):
    """f and the field itself on the nodes of n, for the seed."""
    r = random.Random(seed)
    ax = _axes(n, box)
    e = torch.exp(ax[0]) * torch.exp(ax[1]) * torch.exp(ax[2]) * 0.1
    u = e.clone()
    f = e.mul_(sum(1.0 / v ** 2 for v in box))
    for _ in range(3):
        a, p = r.uniform(0.5, 1.5), [r.randint(1, 3) for _ in range(3)]
        s = [torch.sin(p[d] * math.pi * ax[d]) for d in range(3)]
        k2 = sum((p[d] * math.pi / box[d]) ** 2 for d in range(3))
        t = (s[2] * s[1]) * s[0]
        u.add_(t, alpha=a)
        f.add_(t, alpha=-a * k2)
        del t
    return f, u


def _inner(a):
    return a[1:-1, 1:-1, 1:-1]


def _inputs(n, box, seed):
    f, u = _field(n, box, seed)
    _inner(u).zero_()
    return f, u


def _n(case):
    return (case["nx"], case["ny"], case["nz"])


def _box(case):
    return (case["lx"], case["ly"], case["lz"])


def _problems(case):
    """(n, coarsest, box) of a batch's problems."""
    r = random.Random(case["sizes"])
    out = []
    for _ in range(case["count"]):
        n = tuple(r.choice([32, 48, 64] if case["small"] else [32, 64, 96, 128, 192]) for _ in range(3))
        box = tuple(round(r.uniform(0.7, 1.4) if case["small"] else r.uniform(0.5, 2.0), 3) for _ in range(3))
        out.append((n, tuple(v // (8 if case["small"] else 16) for v in n), box))
    return out


def _target(n, box, seed):
    """The upstream gradient of a misfit to another field: smooth, nonzero on the boundary too."""
    return _field(n, box, seed ^ 0x5A5A5A)[1].sub_(_field(n, box, seed)[1])


def _step_inputs(case, seed):
    n, box = _n(case), _box(case)
    f, u = _field(n, box, seed)
    g = u.clone()
    _inner(g).zero_()
    # coarser solutions as the cascade has them: the field plus an h^4 error
    e = _field(n, box, seed + 101)[1]
    h4 = 1e-7
    u2 = (u + 16 * h4 * e)[::2, ::2, ::2].contiguous()
    u4 = (u + 256 * h4 * e)[::4, ::4, ::4].contiguous()
    return dict(f=f, g=g, u=u.add_(e, alpha=h4), u2=u2, u4=u4)


def prepare(case, seed):
    kind = case["kind"]
    precision = ex.FP32_IR if case["mixed"] else ex.FP64
    if kind == "batch":
        ps = _problems(case)
        solvers = [ex.Solver(n, box, case["tol"], c, precision) for n, c, box in ps]
        fg = [_inputs(n, box, seed * 1009 + i) for i, (n, c, box) in enumerate(ps)]
        ws = torch.empty(ex.batch_workspace_bytes(len(ps)), dtype=torch.uint8, device="cuda")
        return dict(kind=kind, solvers=solvers, f=[v[0] for v in fg], g=[v[1] for v in fg], workspace=ws)
    n, box = _n(case), _box(case)
    if kind == "steps":
        return dict(_step_inputs(case, seed), kind=kind, n=n, box=box)
    f, g = _inputs(n, box, seed)
    s = ex.Solver(n, box, case["tol"], (case["cx"], case["cy"], case["cz"]), precision)
    if case["tuned"]:
        s.autotune()
    st = dict(kind=kind, solver=s, f=f, g=g, ext=case["ext"], grad=case["grad"])
    if kind == "autograd":
        st.update(f=f.requires_grad_(), g=g.requires_grad_(), G=_target(n, box, seed))
    return st


def run(st):
    kind = st["kind"]
    if kind == "batch":
        return ex.solve_batched(st["solvers"], st["f"], st["g"], workspace=st["workspace"])[0]
    if kind == "steps":
        n, box = st["n"], st["box"]
        return dict(b=ex.op_rhs(st["f"], st["g"], n, box), y=ex.op_apply(st["u"], n, box),
                    w=ex.op_exp_finite(st["u2"], st["u4"], st["g"], n), ut=ex.op_exp_true(st["u"], st["u2"], n))
    s = st["solver"]
    if kind == "autograd":
        u = autograd.solve(st["f"], st["g"], s)
        df, dg = torch.autograd.grad(u, (st["f"], st["g"]), st["G"])
        return dict(u=u.detach(), df=df, dg=dg)
    u, ut, _ = s.solve(st["f"], st["g"], want_ext=st["ext"])
    out = dict(u=u)
    if st["ext"]:
        out["ut"] = ut
    if st["grad"]:
        out["ux"], out["uy"], out["uz"] = s.gradient(u)
    return out


def work(case):
    """Inputs read once (f, and g on the boundary) and outputs written once; one application of the operator."""
    if case["kind"] == "batch":
        nodes = sum((n[0] + 1) * (n[1] + 1) * (n[2] + 1) for n, _, _ in _problems(case))
        return dict(bytes=16.0 * nodes, flops=40.0 * nodes)
    n = _n(case)
    nodes = (n[0] + 1) * (n[1] + 1) * (n[2] + 1)
    if case["kind"] == "steps":  # f; u; u_2h and u_4h; u and u_2h read, four arrays written
        return dict(bytes=8.0 * nodes * (3 + 2 / 8 + 1 / 64 + 4), flops=100.0 * nodes)
    if case["kind"] == "autograd":  # f and G read, u, df and dg written
        return dict(bytes=40.0 * nodes, flops=80.0 * nodes)
    arrays = 2 + (1 if case["ext"] else 0) + (3 if case["grad"] else 0)
    return dict(bytes=8.0 * nodes * arrays, flops=40.0 * nodes)


# -------------------------------------------------------------------------------- the exact discrete results
# The discrete system M u = -R f + A_IB g solved directly by sine transforms (dense products in 64 bits), and the
# extrapolations, the compact gradient and the adjoint transposes written out on whole arrays.


def _along(a, mats):
    """mats[d] applied along axis d (x, y, z) of a node array (z, y, x)."""
    x, y, z = mats
    nz, ny, nx = a.shape
    a = (a.reshape(nz * ny, nx) @ x.t().contiguous()).reshape(nz, ny, -1)
    a = (z @ a.reshape(nz, -1)).reshape(z.shape[0], ny, -1)
    return torch.stack([y @ p for p in a.unbind(0)])


def _coef(n, box):
    a, b, c = ((n[d] / box[d]) ** 2 for d in range(3))
    return dict(c0=8 * (a + b + c), x=-(4 * a - b - c), y=-(4 * b - a - c), z=-(4 * c - a - b), xy=-(a + b) / 2,
                xz=-(a + c) / 2, yz=-(b + c) / 2)


def _shift(v, dz, dy, dx):
    nz, ny, nx = (s - 2 for s in v.shape)
    return v[1 + dz:1 + dz + nz, 1 + dy:1 + dy + ny, 1 + dx:1 + dx + nx]


def _apply(v, n, box):
    """M v at the interior nodes, v a node array (its boundary read)."""
    k = _coef(n, box)
    out = k["c0"] * _shift(v, 0, 0, 0)
    for s in (-1, 1):
        out += k["x"] * _shift(v, 0, 0, s) + k["y"] * _shift(v, 0, s, 0) + k["z"] * _shift(v, s, 0, 0)
        for t in (-1, 1):
            out += k["xy"] * _shift(v, 0, s, t) + k["xz"] * _shift(v, s, 0, t) + k["yz"] * _shift(v, s, t, 0)
    return out


def _around(v):
    """R v = (6 v + the six face neighbours) / 2 at the interior nodes."""
    out = 3.0 * _shift(v, 0, 0, 0)
    for s in (-1, 1):
        out += 0.5 * (_shift(v, 0, 0, s) + _shift(v, 0, s, 0) + _shift(v, s, 0, 0))
    return out


def _pad(v):
    return torch.nn.functional.pad(v, (1, 1, 1, 1, 1, 1))


def _edge(g):
    e = g.detach().clone()
    _inner(e).zero_()
    return e


def _direct(b, n, box):
    """M^-1 b on the interior."""
    k = _coef(n, box)
    S, C = [], []
    for d in range(3):
        i = np.arange(1, n[d])
        S.append(torch.from_numpy(np.sin(np.pi * (np.outer(i, i) % (2 * n[d])) / n[d])).cuda())
        C.append(torch.from_numpy(np.cos(np.pi * i / n[d])).cuda())
    X, Y, Z = C[0].reshape(1, 1, -1), C[1].reshape(1, -1, 1), C[2].reshape(-1, 1, 1)
    lam = k["c0"] + 2 * (k["x"] * X + k["y"] * Y + k["z"] * Z) + 4 * (k["xy"] * X * Y + k["xz"] * X * Z + k["yz"] * Y * Z)
    t = _along(b, S)
    t /= lam
    del lam
    t = _along(t, S)
    t *= 8.0 / (n[0] * n[1] * n[2])
    return t


def _discrete(f, g, n, box):
    """The compact scheme's solution on the grid n, with g on the boundary."""
    e = _edge(g)
    u = _pad(_direct(-_around(f) - _apply(e, n, box), n, box))
    return u.add_(e)


def _linear(n):
    """Interpolation from n + 1 nodes to 2 n + 1."""
    m = torch.zeros(2 * n + 1, n + 1, dtype=F64)
    for i in range(n + 1):
        m[2 * i, i] = 1.0
    for i in range(n):
        m[2 * i + 1, i] = m[2 * i + 1, i + 1] = 0.5
    return m.cuda()


def _quartic(n):
    """From n + 1 nodes (n a multiple of 4) to 2 n + 1 by quartic polynomials on cells of four intervals."""
    m = torch.zeros(2 * n + 1, n + 1, dtype=F64)
    for i in range(0, n, 4):
        for t in range(9):
            for q in range(5):
                w = 1.0
                for o in range(5):
                    if o != q:
                        w *= (t / 2 - o) / (q - o)
                m[2 * i + t, i + q] = w
    return m.cuda()


def _ext_true(u, u2, n):
    d = u[::2, ::2, ::2] - u2
    return u + _along(d.contiguous(), [_linear(v // 2) for v in n]) / 15.0


def _ext_finite(u2, u4, g, n):
    d = u2[::2, ::2, ::2] - u4
    w = _along(u2 + _along(d.contiguous(), [_linear(v // 4) for v in n]) / 16.0, [_quartic(v // 2) for v in n])
    e = _edge(g)
    _inner(e).copy_(_inner(w))
    return e


def _derivative(N, h):
    """The fourth-order compact first derivative on N + 1 nodes as a dense matrix."""
    T, B = np.zeros((N + 1, N + 1)), np.zeros((N + 1, N + 1))
    end = np.array([-25.0, 48.0, -36.0, 16.0, -3.0]) / (12.0 * h)
    T[0, 0] = T[N, N] = 1.0
    B[0, :5] = end
    B[N, N - np.arange(5)] = -end
    for i in range(1, N):
        T[i, i - 1], T[i, i], T[i, i + 1] = 1.0, 4.0, 1.0
        B[i, i - 1], B[i, i + 1] = -3.0 / h, 3.0 / h
    return torch.from_numpy(np.linalg.solve(T, B)).cuda()


def _gradient(u, n, box):
    nz, ny, nx = u.shape
    dx, dy, dz = (_derivative(n[d], box[d] / n[d]) for d in range(3))
    ux = (u.reshape(-1, nx) @ dx.t().contiguous()).reshape(u.shape)
    uy = torch.stack([dy @ p for p in u.unbind(0)])
    uz = (dz @ u.reshape(nz, -1)).reshape(u.shape)
    return ux, uy, uz


def _adjoint(G, n, box):
    """dL/df and dL/dg for the upstream gradient G."""
    lam = _pad(_direct(_inner(G).contiguous(), n, box))
    wide = _pad(lam)
    df = -_around(wide)
    e = -_apply(wide, n, box) + G  # A lambda on the boundary nodes: the transposed coupling
    _inner(e).zero_()
    return df, e


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        out = []
        for i, (n, _, box) in enumerate(_problems(case)):
            f, g = _inputs(n, box, seed * 1009 + i)
            out.append(_discrete(f, g, n, box))
        return out
    n, box = _n(case), _box(case)
    if kind == "steps":
        st = _step_inputs(case, seed)
        b = _pad(-_around(st["f"]) - _apply(st["g"], n, box))
        x = _pad(_inner(st["u"]))
        return dict(b=b, y=_pad(_apply(x, n, box)), w=_ext_finite(st["u2"], st["u4"], st["g"], n),
                    ut=_ext_true(st["u"], st["u2"], n))
    f, g = _inputs(n, box, seed)
    u = _discrete(f, g, n, box)
    out = dict(u=u)
    if kind == "autograd":
        out["df"], out["dg"] = _adjoint(_target(n, box, seed), n, box)
        return out
    if case["ext"]:
        m = tuple(v // 2 for v in n)
        u2 = _discrete(f[::2, ::2, ::2].contiguous(), g[::2, ::2, ::2].contiguous(), m, box)
        out["ut"] = _ext_true(u, u2, n)
    if case["grad"]:
        out["ux"], out["uy"], out["uz"] = _gradient(u, n, box)
    return out
