"""Performance cases of the multigrid Wilson-Dirac library.

Each case is one pass through a public entry point of the Python binding, with
everything a user's program keeps (the context with its links, mass and
hierarchy) prepared outside the pass:

  D         ``Context.apply_D``: the Wilson operator on caller fields
  smooth    ``Context.smooth``: MR steps on the fine level from x = 0
  restrict  ``Context.restrict``: P^dagger from the fine level
  prolong   ``Context.prolong``: P to the fine level
  coarse    ``Context.apply_Dc``: the Galerkin operator on the first coarse level
  solve     ``Context.solve``: a multigrid solve on an existing hierarchy
  step      ``Context.mg_setup`` and ``Context.solve``: the benchmark's step
  solve2d   ``Context2d.solve``: the 2d U(1) solve on an existing hierarchy

Sizes are those of the benchmark and the GPU tests (8^4, 16^4, 24^3 x 48, 32^4
and odd-shaped lattices; Nv = 20 and 24; 1 to 32 right-hand sides; 128^2 for
the 2d workload).  Links are ``exp(i eps H)`` and right-hand sides Gaussian, as
in the benchmark; 2d links have von Mises plaquettes at beta = 6.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_0811_4331_amd import qed2d, wdmg

DEV = "cuda:0"
REAL_BYTES = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2}
HALF = ("f16", "bf16")
# Mass of the solves: 0.03 to 0.04 above the critical mass that the benchmark
# uses for fields of this eps (-1.586 to -1.590 at eps 0.45, -0.777 at 0.3),
# which differs little from one field of that eps to another.
EPS, MASS = 0.45, -1.55
SOLVE_TOL = 1e-12
MASS_2D = 0.01


# ---------------------------------------------------------------------------
# The cases
def listed():
    b = {"bx": 4, "by": 4, "bz": 4, "bt": 4}
    l16 = {"lx": 16, "ly": 16, "lz": 16, "lt": 16}
    l24 = {"lx": 24, "ly": 24, "lz": 24, "lt": 48}
    return [
        # one operator application on the smallest lattice of the tests: launches count
        {"name": "D 8^4 f64 1 rhs", "kind": "D", "lx": 8, "ly": 8, "lz": 8, "lt": 8, "nrhs": 1, "prec": "f64"},
        # the operator a Krylov or eigenvalue program calls on a lattice larger than the caches
        {"name": "D 32^4 f64 1 rhs", "kind": "D", "lx": 32, "ly": 32, "lz": 32, "lt": 32, "nrhs": 1, "prec": "f64"},
        # extents that do not cut into 4^4 tiles, an odd batch
        {"name": "D 12x20x10x18 f32 5 rhs", "kind": "D", "lx": 12, "ly": 20, "lz": 10, "lt": 18, "nrhs": 5,
         "prec": "f32"},
        # the benchmark's lattice and batch, the precision of its setup and outer basis
        {"name": "D 24^3x48 f32 32 rhs", "kind": "D", **l24, "nrhs": 32, "prec": "f32"},
        # the smoother as a program of its own (a smoothed source, a preconditioner): a batch of 8
        {"name": "smooth 16^4 f32 8 rhs", "kind": "smooth", **l16, "nrhs": 8, "prec": "f32", "iters": 4},
        # transfers of the benchmark's hierarchy: the V-cycle's storage down, FP32 up
        {"name": "restrict 24^3x48 bf16 32 rhs", "kind": "restrict", **l24, **b, "nv": 24, "nrhs": 32,
         "prec": "bf16"},
        {"name": "prolong 24^3x48 f32 16 rhs", "kind": "prolong", **l24, **b, "nv": 24, "nrhs": 16, "prec": "f32"},
        # coarse operators: the benchmark's first coarse level in its storage, one rhs of the 16^4 workload
        {"name": "coarse 24^3x48 bf16 32 rhs", "kind": "coarse", **l24, **b, "nv": 24, "nrhs": 32, "prec": "bf16"},
        {"name": "coarse 16^4 f64 1 rhs", "kind": "coarse", **l16, **b, "nv": 20, "nrhs": 1, "prec": "f64"},
        # one FP64 solve on a hierarchy in hand (the 16^4 workload)
        {"name": "solve 16^4 f64 1 rhs", "kind": "solve", **l16, **b, "nv": 20, "nrhs": 1, "prec": "f64",
         "iters": 50, "restart": 50},
        # the benchmark's step: FP32 setup, three levels, BF16 V-cycle, a batch
        {"name": "step 24^3x48 bf16 16 rhs", "kind": "step", **l24, **b, "nv": 24, "nv2": 16, "nrhs": 16,
         "prec": "bf16", "iters": 200, "restart": 6},
        # the 2d U(1) workload at its own size
        {"name": "solve2d 128^2", "kind": "solve2d", "lx": 128, "lt": 128, "nv": 8, "nv2": 16, "cycles": 4,
         "iters": 300},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _extents(rng, lo, hi, most):
    """Four extents of lo..hi, any integers, of at most `most` sites."""
    while True:
        d = [_log_int(rng, lo, hi) for _ in range(4)]
        if rng.random() < 0.5:
            d = [max(4, 4 * (x // 4)) for x in d]
        if d[0] * d[1] * d[2] * d[3] <= most:
            return dict(zip(("lx", "ly", "lz", "lt"), d))


def draw(rng):
    kind = rng.choice(["D", "D", "D", "smooth", "smooth", "restrict", "restrict", "prolong", "prolong", "coarse",
                       "coarse", "solve", "step", "solve2d"])
    if kind == "D":
        c = {"kind": kind, **_extents(rng, 4, 40, 1 << 20), "prec": rng.choice(["f64", "f32", "f32"])}
        vol = c["lx"] * c["ly"] * c["lz"] * c["lt"]
        c["nrhs"] = _log_int(rng, 1, max(1, min(32, (1 << 24) // vol)))
        return c
    if kind == "smooth":
        c = {"kind": kind, **_extents(rng, 6, 24, 1 << 18), "prec": rng.choice(["f64", "f32", "f32"])}
        c["nrhs"], c["iters"] = _log_int(rng, 1, 16), rng.randint(1, 6)
        return c
    if kind in ("restrict", "prolong", "coarse"):
        # aggregates of the tests and the benchmark: 4^4, some smaller ones, odd ones among them
        blk = [4] * 4 if rng.random() < 0.6 else [rng.choice([2, 3, 4]) for _ in range(4)]
        while True:
            n = [rng.randint(2, 8) for _ in range(4)]
            d = [x * y for x, y in zip(blk, n)]
            if d[0] * d[1] * d[2] * d[3] <= 1 << 19:
                break
        nv = rng.randint(8, 32)
        nv = min(nv, 6 * blk[0] * blk[1] * blk[2] * blk[3] // 2)
        precs = {"restrict": ["f64", "f32", "bf16", "f16"], "prolong": ["f64", "f32", "f32"],
                 "coarse": ["f64", "f32", "bf16", "f16"]}[kind]
        return {"kind": kind, **dict(zip(("lx", "ly", "lz", "lt"), d)), **dict(zip(("bx", "by", "bz", "bt"), blk)),
                "nv": nv, "nrhs": _log_int(rng, 1, 32), "prec": rng.choice(precs)}
    b = {"bx": 4, "by": 4, "bz": 4, "bt": 4}
    if kind == "solve":
        d = [rng.choice([8, 12, 16]) for _ in range(4)]
        return {"kind": kind, **dict(zip(("lx", "ly", "lz", "lt"), d)), **b, "nv": rng.randint(12, 24),
                "nrhs": _log_int(rng, 1, 12), "prec": rng.choice(["f64", "f32", "bf16"]),
                "iters": rng.choice([30, 50, 80]), "restart": rng.choice([16, 32, 50])}
    if kind == "step":
        d = [rng.choice([16, 24]) for _ in range(3)] + [rng.choice([16, 24, 32])]
        return {"kind": kind, **dict(zip(("lx", "ly", "lz", "lt"), d)), **b, "nv": rng.choice([16, 20, 24]),
                "nv2": rng.choice([12, 16]), "nrhs": rng.randint(4, 16), "prec": rng.choice(["bf16", "bf16", "f32"]),
                "iters": rng.choice([100, 200]), "restart": rng.choice([6, 8, 12])}
    d = [rng.choice([48, 64, 80, 96, 112, 128]) for _ in range(2)]
    return {"kind": kind, "lx": d[0], "lt": d[1], "nv": rng.choice([6, 8, 10]), "nv2": rng.choice([8, 12, 16]),
            "cycles": rng.choice([1, 4]), "iters": rng.choice([100, 200, 300])}


# ---------------------------------------------------------------------------
# Inputs, from the seed alone
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _dims(case):
    return case["lx"], case["ly"], case["lz"], case["lt"]


def _cdtype(prec):
    return torch.complex128 if prec == "f64" else torch.complex64


def _links(dims, eps, gen):
    """exp(i eps H) per link, H traceless Hermitian with N(0,1) entries; [t,z,y,x,4,3,3]."""
    lx, ly, lz, lt = dims
    n = lx * ly * lz * lt * 4
    diag = torch.randn((n, 3), generator=gen, device=DEV, dtype=torch.float64)
    off = torch.randn((n, 3, 2), generator=gen, device=DEV, dtype=torch.float64)
    h = torch.zeros((n, 3, 3), device=DEV, dtype=torch.complex128)
    for a in range(3):
        h[:, a, a] = diag[:, a] - diag.mean(1)
    for k, (a, b) in enumerate(((0, 1), (0, 2), (1, 2))):
        z = torch.complex(off[:, k, 0], off[:, k, 1])
        h[:, a, b] = z
        h[:, b, a] = z.conj()
    # the exponential as (Taylor of H / 16) ^ 16, brought back onto SU(3)
    m = (1j * eps / 16) * h
    del h
    u = torch.eye(3, device=DEV, dtype=torch.complex128) + m
    term = m
    for k in range(2, 9):
        term = _mul3(term, m) / k
        u = u + term
    for _ in range(4):
        u = _mul3(u, u)
    r0 = u[:, 0] / torch.linalg.vector_norm(u[:, 0], dim=1, keepdim=True)
    r1 = u[:, 1] - (r0.conj() * u[:, 1]).sum(1, keepdim=True) * r0
    r1 = r1 / torch.linalg.vector_norm(r1, dim=1, keepdim=True)
    r2 = torch.stack([r0[:, 1] * r1[:, 2] - r0[:, 2] * r1[:, 1], r0[:, 2] * r1[:, 0] - r0[:, 0] * r1[:, 2],
                      r0[:, 0] * r1[:, 1] - r0[:, 1] * r1[:, 0]], 1).conj()
    return torch.stack([r0, r1, r2], 1).reshape(lt, lz, ly, lx, 4, 3, 3).contiguous()


def _mul3(a, b):
    return sum(a[:, :, k, None] * b[:, None, k, :] for k in range(3))


def _gauss(shape, gen, dtype):
    return torch.randn(shape, generator=gen, device=DEV, dtype=dtype)


def _inputs(case, seed):
    """Links, mass and the tensors of a 4d case."""
    gen = _gen(seed)
    lx, ly, lz, lt = _dims(case)
    kind, nrhs = case["kind"], case["nrhs"]
    fine = (lt, lz, ly, lx, 4, 3)
    dt = torch.complex128 if kind in ("solve", "step") else _cdtype(case["prec"])
    i = {"U": _links((lx, ly, lz, lt), EPS, gen)}
    if "nv" in case:
        i["V"] = _gauss((case["nv"],) + fine, gen, torch.complex128)
        crs = (lt // case["bt"], lz // case["bz"], ly // case["by"], lx // case["bx"], 2, case["nv"])
        if "nv2" in case:
            i["V2"] = _gauss((case["nv2"],) + crs, gen, torch.complex128)
    shape = (nrhs,) + (crs if kind in ("prolong", "coarse") else fine)
    i["b"] = _gauss(shape, gen, dt)
    return i


def _level(case, i):
    return {"block": (case["bx"], case["by"], case["bz"], case["bt"]), "nv": case["nv"], "vectors": i["V"],
            "setup_iters": case.get("iters", 0), "setup_prec": "f64" if case["prec"] == "f64" else "f32"}


def _inputs2d(case, seed):
    """2d links with von Mises plaquettes (beta 6), candidates and a right-hand side."""
    rng = np.random.default_rng(int(seed))
    lx, lt = case["lx"], case["lt"]
    th0, th1 = np.zeros((lt, lx)), np.zeros((lt, lx))
    plaq = rng.vonmises(0.0, 6.0, (lt, lx))
    th0[0] = rng.uniform(-np.pi, np.pi, lx)
    for t in range(lt - 1):
        th0[t + 1] = th0[t] - plaq[t]
    # the last row's t links close its plaquettes but one
    th1[lt - 1, 1:] = np.cumsum(plaq[lt - 1, :-1] - (th0[lt - 1] - th0[0])[:-1])
    g = rng.uniform(-np.pi, np.pi, (lt, lx))
    th0 += g - np.roll(g, -1, 1)
    th1 += g - np.roll(g, -1, 0)
    u = torch.from_numpy(np.exp(1j * np.stack([th0, th1], -1))).to(DEV)
    gen = _gen(seed)
    v = [_gauss((case["nv"], lt, lx, 2, 1), gen, torch.complex128),
         _gauss((case["nv2"], lt // 4, lx // 4, 2, case["nv"]), gen, torch.complex128)]
    return {"U": u, "V": v, "b": _gauss((lt, lx, 2), gen, torch.complex128)}


def prepare(case, seed):
    kind = case["kind"]
    if kind == "solve2d":
        i = _inputs2d(case, seed)
        ctx = qed2d.Context2d((case["lx"], case["lt"]), DEV)
        ctx.set_gauge(i["U"], -1)
        ctx.set_mass(MASS_2D)
        ctx.mg_setup([case["nv"], case["nv2"]], i["V"], setup_iters=case["iters"], coarse_cycles=case["cycles"])
        return {"case": case, "ctx": ctx, "b": i["b"]}
    i = _inputs(case, seed)
    ctx = wdmg.Context(_dims(case), DEV)
    ctx.set_gauge(i["U"], -1)
    ctx.set_mass(MASS)
    s = {"case": case, "ctx": ctx, "b": i["b"]}
    if kind == "step":
        s["levels"] = [_level(case, i), {"block": (2, 2, 2, 2), "nv": case["nv2"], "vectors": i["V2"],
                                         "setup_iters": 25, "setup_prec": "f32"}]
    elif "nv" in case:
        ctx.mg_setup([_level(case, i)], coarse_tol=0.1, use_alpha=False)
    return s


def run(s):
    case, ctx, b = s["case"], s["ctx"], s["b"]
    kind = case["kind"]
    if kind == "D":
        return ctx.apply_D(b, prec=case["prec"])
    if kind == "smooth":
        return ctx.smooth(0, torch.zeros_like(b), b, case["iters"], prec=case["prec"])
    if kind == "restrict":
        return ctx.restrict(0, b, prec=case["prec"])
    if kind == "prolong":
        return ctx.prolong(0, b, prec=case["prec"])
    if kind == "coarse":
        return ctx.apply_Dc(1, b, prec=case["prec"])
    if kind == "solve2d":
        return ctx.solve(b, method="mg-bicgstab", tol=SOLVE_TOL)[0]
    if kind == "step":
        ctx.mg_setup(s["levels"], coarse_tol=0.3, use_alpha=False)
    return ctx.solve(b, tol=SOLVE_TOL, restart=case["restart"], mg_prec=case["prec"])[0]


def work(case):
    """Each input once and each output once in the pass's own precision (links
    as the two rows that determine them); operations of the operator sums.  Of
    a solve: its right-hand sides, solutions and candidates, and ten V-cycles'
    worth of operator applications, which the fastest case takes."""
    kind = case["kind"]
    if kind == "solve2d":
        vol = case["lx"] * case["lt"]
        return {"bytes": vol * (2 * 32 + 32 + 16 * 2 * case["nv"]), "flops": vol * 8 * 18 * 60}
    lx, ly, lz, lt = _dims(case)
    vol, nrhs, rb = lx * ly * lz * lt, case["nrhs"], REAL_BYTES[case["prec"]]
    io = 16 if case["prec"] == "f64" else 8  # bytes of a complex number at the boundary
    if kind == "D":
        return {"bytes": vol * (24 * io * nrhs + 48 * rb), "flops": 1368 * vol * nrhs}
    if kind == "smooth":
        return {"bytes": vol * (24 * io * nrhs + 48 * rb), "flops": (1368 + 192) * vol * nrhs * case["iters"]}
    nv = case["nv"]
    agg = vol // (case["bx"] * case["by"] * case["bz"] * case["bt"])
    if kind in ("restrict", "prolong"):
        return {"bytes": vol * 12 * (io * nrhs + 2 * rb * nv) + agg * 2 * nv * io * nrhs, "flops": 96 * vol * nv * nrhs}
    if kind == "coarse":
        return {"bytes": agg * (9 * 4 * nv * nv * 2 * rb + 2 * 2 * nv * io * nrhs),
                "flops": agg * 72 * 4 * nv * nv * nrhs}
    setup = case["iters"] * nv if kind == "step" else 0
    return {"bytes": vol * (24 * 16 * nrhs + 48 * 8 + 12 * 16 * nv), "flops": 1368 * vol * (60 * nrhs + setup)}


# ---------------------------------------------------------------------------
# The same in 64 bits, from the operator's definition
def _hop(u, psi, mu, step):
    """(1 -+ gamma_mu) U psi(x +- mu) on [..., t, z, y, x, 4, 3], antiperiodic in t."""
    ax = {0: -3, 1: -4, 2: -5, 3: -6}[mu]
    f = torch.roll(psi, -step, ax)
    link = u[..., mu, :, :]
    if step < 0:
        link = torch.roll(link, 1, ax).conj().transpose(-1, -2)  # [t,z,y,x,3,3]: its axes -6.. are psi's
    if mu == 3:
        f = f.clone()
        f[..., -1 if step > 0 else 0, :, :, :, :, :] *= -1
    p = f.unbind(-2)
    if mu == 0:
        g = (-1j * p[3], -1j * p[2], 1j * p[1], 1j * p[0])
    elif mu == 1:
        g = (-p[3], p[2], p[1], -p[0])
    elif mu == 2:
        g = (-1j * p[2], 1j * p[3], 1j * p[0], -1j * p[1])
    else:
        g = (p[2], p[3], p[0], p[1])
    h = torch.stack([a - step * b for a, b in zip(p, g)], -2)
    return sum(link[..., None, :, k] * h[..., k, None] for k in range(3))


def _D(u, psi, m):
    """The Wilson operator on one field or a batch, one field at a time."""
    if psi.dim() > 6:
        return torch.stack([_D(u, f, m) for f in psi])
    out = (4.0 + m) * psi
    for mu in range(4):
        for step in (1, -1):
            out = out - 0.5 * _hop(u, psi, mu, step)
    return out


def _dots(a, b):
    return (a.conj() * b).reshape(a.shape[0], -1).sum(1)


def _to_blocks(f, case):
    """[n, t, z, y, x, 4, 3] -> [aggregate (t,z,y,x), chirality, row, n]."""
    n, lt, lz, ly, lx = f.shape[:5]
    bx, by, bz, bt = case["bx"], case["by"], case["bz"], case["bt"]
    f = f.reshape(n, lt // bt, bt, lz // bz, bz, ly // by, by, lx // bx, bx, 2, 6)
    f = f.permute(1, 3, 5, 7, 9, 2, 4, 6, 8, 10, 0)
    return f.reshape(-1, 2, bt * bz * by * bx * 6, n)


def _from_blocks(q, case):
    lx, ly, lz, lt = _dims(case)
    bx, by, bz, bt = case["bx"], case["by"], case["bz"], case["bt"]
    n = q.shape[-1]
    q = q.reshape(lt // bt, lz // bz, ly // by, lx // bx, 2, bt, bz, by, bx, 6, n)
    return q.permute(10, 0, 5, 1, 6, 2, 7, 3, 8, 4, 9).reshape(n, lt, lz, ly, lx, 4, 3)


def _block_q(v, case):
    """Orthonormal columns of every (aggregate, chirality) block, diag(R) > 0."""
    q = _to_blocks(v, case).clone()
    for j in range(q.shape[-1]):
        for _ in range(2):
            if j:
                c = torch.matmul(q[..., :j].transpose(-1, -2).conj().contiguous(), q[..., j:j + 1].contiguous())
                q[..., j:j + 1] -= torch.matmul(q[..., :j].contiguous(), c)
        q[..., j] /= torch.linalg.vector_norm(q[..., j], dim=-1, keepdim=True)
    return q


def _restrict(q, f, case):
    """[n, fine] -> [n, t, z, y, x, 2, nv]."""
    lx, ly, lz, lt = _dims(case)
    c = torch.matmul(q.transpose(-1, -2).conj().contiguous(), _to_blocks(f, case).contiguous())
    c = c.reshape(lt // case["bt"], lz // case["bz"], ly // case["by"], lx // case["bx"], 2, q.shape[-1], f.shape[0])
    return c.permute(6, 0, 1, 2, 3, 4, 5).contiguous()


def _prolong(q, c, case):
    cc = c.permute(1, 2, 3, 4, 5, 6, 0).reshape(-1, 2, c.shape[-1], c.shape[0]).contiguous()
    return _from_blocks(torch.matmul(q, cc), case)


def _solve(apply, b, tol=3e-14, maxit=4000):
    """BiCGStab per right-hand side, restarted from the true residual, to ||b - A x|| <= tol ||b||."""
    x, bn = torch.zeros_like(b), torch.linalg.vector_norm(b)
    it = 0
    while it < maxit:
        r = b - apply(x)
        if torch.linalg.vector_norm(r) <= tol * bn:
            return x
        rh, p, rho = r.clone(), r.clone(), torch.vdot(r.reshape(-1), r.reshape(-1))
        r0 = torch.linalg.vector_norm(r)
        while it < maxit:
            it += 1
            v = apply(p)
            al = rho / torch.vdot(rh.reshape(-1), v.reshape(-1))
            s = r - al * v
            t = apply(s)
            om = torch.vdot(t.reshape(-1), s.reshape(-1)) / torch.vdot(t.reshape(-1), t.reshape(-1))
            x = x + al * p + om * s
            r = s - om * t
            new = torch.vdot(rh.reshape(-1), r.reshape(-1))
            p = r + (new / rho) * (al / om) * (p - om * v)
            rho = new
            if it % 16 == 0 and (torch.linalg.vector_norm(r) <= 0.5 * tol * bn
                                 or torch.linalg.vector_norm(r) <= 1e-5 * r0):
                break
    return x


def _D2(u, psi, m):
    out = (2.0 + m) * psi
    for mu, ax in ((0, -2), (1, -3)):
        for step in (1, -1):
            f = torch.roll(psi, -step, ax)
            link = u[..., mu] if step > 0 else torch.roll(u[..., mu], 1, 1 - mu).conj()
            if mu == 1:
                f[-1 if step > 0 else 0] *= -1
            p0, p1 = f[..., 0], f[..., 1]
            g = (p1, p0) if mu == 0 else (-1j * p1, 1j * p0)
            h = torch.stack([p0 - step * g[0], p1 - step * g[1]], -1)
            out = out - 0.5 * link[..., None] * h
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "solve2d":
        i = _inputs2d(case, seed)
        return _solve(lambda f: _D2(i["U"], f, MASS_2D), i["b"], maxit=20000)
    if kind == "step" or kind == "solve" and case["lx"] * case["ly"] * case["lz"] * case["lt"] * case["nrhs"] > 1 << 17:
        return None
    i = _inputs(case, seed)
    u, b = i["U"], i["b"].to(torch.complex128)
    if kind == "D":
        return _D(u, b, MASS)
    if kind == "smooth":
        x, r = torch.zeros_like(b), b.clone()
        for _ in range(case["iters"]):
            p = _D(u, r, MASS)
            a = (0.8 * _dots(p, r) / _dots(p, p)).reshape(-1, 1, 1, 1, 1, 1, 1)
            x, r = x + a * r, r - a * p
        return x
    if kind == "solve":
        return torch.stack([_solve(lambda f: _D(u, f, MASS), f) for f in b])
    q = _block_q(i["V"], case)
    if kind == "restrict":
        return _restrict(q, b, case)
    if kind == "prolong":
        return _prolong(q, b, case)
    out = []
    for f in b:
        out.append(_restrict(q, _D(u, _prolong(q, f[None], case), MASS), case)[0])
    return torch.stack(out)
