"""What callers may do with their own buffers: input and output that overlap
give what separate buffers give, to the last bit."""
import numpy as np
import pytest
import torch

import synthetic
from paper_0811_4331_amd import wdmg

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
DIMS, BLK, NV = (8, 4, 4, 8), (4, 4, 4, 4), 6


def gpu(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


@pytest.fixture(scope="module")
def ctx():
    lx, ly, lz, lt = DIMS
    c = wdmg.Context(DIMS, DEV)
    c.set_gauge(gpu(synthetic.gauge_field(DIMS, 0.35, 981)), t_bc=-1)
    c.set_mass(-0.4)
    v = synthetic.gaussian_vectors((NV, lt, lz, ly, lx, 4, 3), 982)
    c.mg_setup([{"block": BLK, "nv": NV, "setup_iters": 0, "vectors": gpu(v)}])
    yield c
    c.close()


def overlapping(src, out_shape, shift):
    """`src` copied into one allocation and an output of `out_shape` that starts
    `shift` numbers after it (before it for a negative shift)."""
    n = int(np.prod(out_shape))
    flat = torch.zeros(src.numel() + n + 2 * abs(shift), dtype=src.dtype, device=DEV)
    a = max(0, -shift)
    x = flat[a:a + src.numel()].view(src.shape)
    x.copy_(src)
    out = flat[a + shift:a + shift + n].view(out_shape)
    return x, out


def call(ctx, name, *args):
    ctx._check(getattr(ctx.lib, name)(ctx.h, *args))


@pytest.mark.parametrize("shift", [4, -10, 6145, 0])
@pytest.mark.parametrize("prec", ["f64", "f32", "bf16"])
def test_input_and_output_may_overlap(ctx, prec, shift):
    nrhs, p = 3, wdmg.PREC[prec]
    dt = np.complex128 if prec == "f64" else np.complex64
    f = gpu(synthetic.gaussian_spinor(DIMS, seed=983, nrhs=nrhs).astype(dt))
    coarse = ctx.restrict(0, f, prec=prec)
    if shift:  # the same pointer is refused here
        ref = ctx.apply_D(f, prec=prec)
        x, out = overlapping(f, f.shape, shift)
        assert torch.equal(ctx.apply_D(x, prec=prec, out=out), ref)
        if prec != "bf16":
            x, out = overlapping(f, f.shape, shift)
            assert torch.equal(ctx.apply_D_noalloc(x, out, prec=prec), ref)
        x, out = overlapping(f, f.shape, shift)
        ref = ctx.roundtrip(f, prec=prec)
        call(ctx, "wdmg_roundtrip", out.data_ptr(), x.data_ptr(), nrhs, p)
        assert torch.equal(out, ref)
    x, out = overlapping(f, coarse.shape, max(shift, 0))
    call(ctx, "wdmg_restrict", 0, out.data_ptr(), x.data_ptr(), nrhs, p)
    assert torch.equal(out, coarse)
    ref = ctx.prolong(0, coarse, prec=prec)
    x, out = overlapping(coarse, f.shape, min(shift, 0))
    call(ctx, "wdmg_prolong", 0, out.data_ptr(), x.data_ptr(), nrhs, p)
    assert torch.equal(out, ref)


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_smoothing_where_a_solution_is_the_next_right_hand_side(ctx, prec):
    """x one field after b: each right-hand side is smoothed before the next is
    read, so the sequence is that of single calls."""
    dt = np.complex128 if prec == "f64" else np.complex64
    n = int(np.prod(ctx.fine_shape()))
    b = gpu(synthetic.gaussian_spinor(DIMS, seed=984, nrhs=4).astype(dt))
    flat = b.reshape(-1).clone()
    for j in range(3):
        ctx.smooth(0, flat[(j + 1) * n:(j + 2) * n].view(b.shape[1:]), flat[j * n:(j + 1) * n].view(b.shape[1:]), 3,
                   prec=prec)
    both = b.reshape(-1).clone()
    ctx.smooth(0, both[n:].view((3,) + b.shape[1:]), both[:3 * n].view((3,) + b.shape[1:]), 3, prec=prec)
    assert torch.equal(both, flat)


@pytest.mark.parametrize("prec", ["f16", "bf16"])
def test_smoothing_of_very_many_right_hand_sides(prec):
    """The largest batch, far beyond the 64 that there are step-size scalars for:
    each right-hand side gets its own steps, and a solve after it gives what it
    gave before."""
    dims = (4, 4, 4, 4)
    ctx = wdmg.Context(dims, DEV)
    ctx.set_gauge(gpu(synthetic.gauge_field(dims, 0.35, 985)), t_bc=-1)
    ctx.set_mass(-0.2)
    v = synthetic.gaussian_vectors((4,) + ctx.fine_shape(), 986)
    v2 = synthetic.gaussian_vectors((4, 2, 2, 2, 2, 2, 4), 987)
    ctx.mg_setup([{"block": (2, 2, 2, 2), "nv": 4, "setup_iters": 10, "vectors": gpu(v)},
                  {"block": (2, 2, 1, 1), "nv": 4, "setup_iters": 10, "vectors": gpu(v2)}], coarse_tol=1e-2)
    b = gpu(synthetic.gaussian_spinor(dims, seed=988, nrhs=2))
    before, st = ctx.solve(b, tol=1e-10, restart=20, maxit=200)
    assert all(s["converged"] for s in st)
    n = 65535
    f = torch.zeros((n,) + ctx.fine_shape(), dtype=torch.complex64, device=DEV)
    for j in (0, 63, 64, n - 1):
        f[j] = b[j % 2]
    x = ctx.smooth(0, torch.zeros_like(f), f, 3, prec=prec)
    for j in (0, 63, 64, n - 1):
        one = ctx.smooth(0, torch.zeros_like(f[j]), f[j].clone(), 3, prec=prec)
        assert float((x[j] - one).abs().max() / one.abs().max()) < 1e-2  # 16-bit roundings of another form
    assert not x[1:63].any() and not x[65:n - 1].any()
    after, st2 = ctx.solve(b, tol=1e-10, restart=20, maxit=200)
    assert torch.equal(before, after) and [s["iters"] for s in st] == [s["iters"] for s in st2]
    ctx.close()
