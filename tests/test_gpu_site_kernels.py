"""The kernels that work on fields as the caller lays them out, at the sizes
where they can go wrong: the tile form of the Wilson operator over more tiles
than workgroups and over lattices of a few tiles, the matrix-core transfers at
the edges of their column and right-hand-side tiles and on aggregates that are
no whole number of their units, buffers that are aligned to a complex number
only, and the block QR's row counts.

Tolerances: u = 2^-24.  A Wilson result sums 8 x 3 complex products per
component of numbers of magnitude about 1: 1e-6 of the largest result covers
FP32, 1e-13 FP64.  A transfer's element sums n complex products; with rounding
errors of either sign its error is at most (4 sqrt(2 n) + 1) u times the sum
of the products' magnitudes (n = rows of an aggregate's chirality down, Nv
up), and 2^-53 in place of u in FP64."""
import numpy as np
import pytest
import torch

import synthetic
from oracle import precision, transfer, wilson
from paper_0811_4331_amd import wdmg

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def gpu(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


def rel(a, b):
    return float(np.abs(a - b).max() / np.abs(b).max())


def context(dims, seed, m=-0.4):
    u = synthetic.gauge_field(dims, 0.35, seed)
    ctx = wdmg.Context(dims, DEV)
    ctx.set_gauge(gpu(u), t_bc=-1)
    ctx.set_mass(m)
    return ctx, u


@pytest.mark.parametrize("dims,nrhs", [((16, 16, 16, 20), 2),  # 320 tiles: a whole round and a shared one
                                       ((4, 4, 4, 12), 5),     # three tiles, each its own x, y, z neighbour
                                       ((4, 4, 4, 4), 3)])     # one tile, its own neighbour everywhere
def test_tile_form_over_all_its_work(dims, nrhs):
    ctx, u = context(dims, 901)
    psi = synthetic.gaussian_spinor(dims, seed=902, nrhs=nrhs).astype(np.complex64)
    ctx.set_tuning("dslash", 5)
    out = ctx.apply_D(gpu(psi), prec="f32").cpu().numpy()
    ctx.set_tuning("dslash", 1)
    other = ctx.apply_D(gpu(psi), prec="f32").cpu().numpy()
    assert rel(out, other) < 1e-6
    for j in {0, nrhs - 1}:
        assert rel(out[j], wilson.apply_D(u, psi[j].astype(np.complex128), -0.4, -1.0)) < 1e-6
    ctx.close()


def _hierarchy(dims, blk, nv, seed):
    ctx, u = context(dims, seed)
    lx, ly, lz, lt = dims
    v = synthetic.gaussian_vectors((nv, lt, lz, ly, lx, 4, 3), seed + 1)
    ctx.mg_setup([{"block": blk, "nv": nv, "setup_iters": 0, "vectors": gpu(v)}])
    q, _ = transfer.block_orthonormalize(transfer.as_chiral(v), blk)
    return ctx, q


@pytest.mark.parametrize("prec", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("dims,blk,nv,nrhs", [
    ((8, 4, 4, 4), (4, 4, 4, 4), 16, 2),    # one full column tile
    ((8, 4, 4, 4), (4, 4, 4, 4), 17, 16),   # one column into the second; a full rhs tile
    ((4, 4, 4, 8), (4, 4, 4, 4), 32, 17),   # both column tiles full, one rhs into the second tile
    ((4, 4, 8, 4), (4, 4, 4, 4), 1, 33),    # one column, a third rhs tile
    ((4, 4, 4, 4), (2, 2, 2, 2), 7, 3),     # 16-site aggregates: one unit
    ((6, 4, 4, 4), (3, 2, 2, 2), 9, 4),     # 24 sites: no whole number of 16-site units
    ((6, 6, 3, 2), (3, 3, 3, 2), 5, 2),     # 54 sites: neither 8 nor 16 divides them
    ((4, 4, 4, 8), (4, 4, 4, 4), 20, 1),    # one right-hand side
])
def test_transfers_at_tile_edges(prec, dims, blk, nv, nrhs):
    ctx, q = _hierarchy(dims, blk, nv, 911 + nv)
    cdt = np.complex128 if prec == "f64" else np.complex64
    unit = 2.0 ** (-53 if prec == "f64" else -24)
    f = synthetic.gaussian_spinor(dims, seed=921, nrhs=nrhs).astype(cdt)
    rows = 6 * int(np.prod(blk))
    qs, fs = q, f.astype(np.complex128)
    if prec in ("f16", "bf16"):  # the operator acts on what 16-bit storage holds
        q32 = precision.round_f32(q)
        qs = (precision.round_16(q32.real, prec) + 1j * precision.round_16(q32.imag, prec)).astype(np.complex128)
        fs = np.stack([precision.store_fine(x.astype(np.complex128), prec) for x in f]).astype(np.complex128)
    # the first 2 for the FP64 prolongator's own rounding and the FP32 copy
    down, up = (unit * (4 * np.sqrt(2 * n) + 2) for n in (rows, nv))
    got = ctx.restrict(0, gpu(f), prec=prec).cpu().numpy().astype(np.complex128)
    for j in range(nrhs):
        fc = transfer.as_chiral(fs[j])
        ref, mag = transfer.restrict(qs, fc, blk), np.abs(transfer.restrict(np.abs(qs), np.abs(fc), blk))
        assert np.all(np.abs(got[j] - ref) <= down * mag + 1e-13), (j, float(np.abs(got[j] - ref).max()))
    c = synthetic.gaussian_vectors((nrhs,) + got.shape[1:], 931).astype(cdt)
    back = ctx.prolong(0, gpu(c), prec=prec).cpu().numpy().astype(np.complex128)
    for j in range(nrhs):
        cc = c[j].astype(np.complex128)
        ref = transfer.as_spinor(transfer.prolong(qs, cc, blk))
        mag = np.abs(transfer.as_spinor(transfer.prolong(np.abs(qs), np.abs(cc), blk)))
        tol = up * mag + 1e-13
        if prec in ("f16", "bf16"):  # stored with a site scale
            top = np.maximum(np.abs(ref.real), np.abs(ref.imag)).max(axis=(-2, -1), keepdims=True)
            tol = tol + 2 * precision.HALF_ULP[prec] * top
        assert np.all(np.abs(back[j] - ref) <= tol), (j, float(np.abs(back[j] - ref).max()))
    ctx.close()


@pytest.mark.parametrize("dims,blk,nv", [((4, 4, 4, 4), (2, 2, 1, 1), 6),    # 24 rows
                                         ((6, 6, 6, 4), (6, 6, 3, 2), 8),    # 648 rows: three per thread
                                         ((8, 8, 4, 8), (8, 8, 4, 2), 5)])   # 3072 rows: more than registers hold
def test_block_qr_row_counts(dims, blk, nv):
    ctx, q = _hierarchy(dims, blk, nv, 941)
    got = ctx.get_prolongator(0).cpu().numpy().reshape(q.shape)
    assert rel(got, q) < 1e-12
    ctx.close()


def test_buffers_aligned_to_one_number():
    """Complex64 buffers that start 8 bytes off a 16-byte boundary give what
    aligned ones give."""
    dims, blk, nv, nrhs = (8, 4, 4, 8), (4, 4, 4, 4), 6, 3
    ctx, _ = _hierarchy(dims, blk, nv, 951)

    def off(t):  # the same values, 8 bytes into an allocation
        flat = torch.empty(t.numel() + 1, dtype=t.dtype, device=DEV)
        flat[1:] = t.reshape(-1)
        out = flat[1:].view(t.shape)
        assert out.data_ptr() % 16 == 8
        return out

    psi = gpu(synthetic.gaussian_spinor(dims, seed=952, nrhs=nrhs).astype(np.complex64))
    for prec in ("f32", "bf16"):
        out = off(torch.zeros_like(psi))
        ctx.apply_D(off(psi), prec=prec, out=out)
        assert torch.equal(out, ctx.apply_D(psi, prec=prec))
        x0 = ctx.smooth(0, torch.zeros_like(psi), psi, 2, prec=prec)
        assert torch.equal(ctx.smooth(0, off(torch.zeros_like(psi)), off(psi), 2, prec=prec), x0)
        c = ctx.restrict(0, psi, prec=prec)
        assert torch.equal(ctx.restrict(0, off(psi), prec=prec), c)
        assert torch.equal(ctx.prolong(0, off(c), prec=prec), ctx.prolong(0, c, prec=prec))
    out = off(torch.zeros_like(psi))
    ctx.apply_D_noalloc(off(psi), out, prec="f32")
    assert torch.equal(out, ctx.apply_D(psi, prec="f32"))
    ctx.close()


@pytest.mark.parametrize("dims,blk,nv,nrhs", [
    ((4, 4, 4, 4), (2, 2, 2, 2), 1, 2),       # two rows; the sites are each other's neighbours
    ((8, 8, 4, 8), (4, 4, 4, 4), 8, 16),      # one whole row tile, one whole tile of right-hand sides
    ((8, 8, 8, 8), (4, 4, 4, 4), 9, 17),      # one row, one column and one right-hand side over
    ((8, 8, 8, 16), (4, 4, 4, 4), 32, 33),    # the most rows
    ((16, 16, 16, 16), (2, 2, 2, 4), 5, 35),  # sites enough for two tiles per workgroup, the last one ragged
    ((8, 12, 12, 20), (2, 2, 2, 2), 3, 16),   # 720 sites: three waves, one tile
])
def test_batched_coarse_operator_at_tile_edges(dims, blk, nv, nrhs):
    """A batch on the matrix cores against one right-hand side at a time on the
    vector units.  Both sum 9 x 2 Nv <= 576 complex products: 2e-6 (1e-13 in
    FP64) of the largest result covers either order.  With 16-bit blocks the
    batch also rounds its vectors, by at most one half unit of the column's
    largest number each: errors of random sign, under 16 half units of the
    largest result."""
    ctx, _ = context(dims, 931)
    lx, ly, lz, lt = dims
    v = synthetic.gaussian_vectors((nv, lt, lz, ly, lx, 4, 3), 930)
    ctx.mg_setup([{"block": blk, "nv": nv, "setup_iters": 0, "vectors": gpu(v)}])
    c = synthetic.gaussian_vectors((nrhs,) + tuple(ctx.coarse_shape(1)), 932)
    for prec, tol in (("f64", 1e-13), ("f32", 2e-6), ("bf16", 16 * precision.HALF_ULP["bf16"]),
                      ("f16", 16 * precision.HALF_ULP["f16"])):
        v = gpu(c if prec == "f64" else c.astype(np.complex64))
        out = ctx.apply_Dc(1, v, prec=prec).cpu().numpy()
        for j in range(nrhs):
            one = ctx.apply_Dc(1, v[j], prec=prec).cpu().numpy()
            assert rel(out[j], one) < tol, (prec, j)
    ctx.close()


@pytest.mark.parametrize("dims,nvs,cycles", [
    ((20, 28), [3], 1),       # 6 dof per site: the general stencil, its sums in a launch of their own
    ((24, 40), [4], 1),       # 8 dof; fields of 1920 numbers end inside a workgroup
    ((24, 40), [16], 1),      # 32 dof
    ((48, 48), [8, 4], 3),    # repeated coarse cycles
    ((272, 272), [8, 4], 2),  # 68^2 sites of 16 dof: more workgroups than the update adds up
])
def test_2d_cycles_with_the_sums_in_the_operator(dims, nvs, cycles):
    """The multigrid cycle of the 2d workload where its MR steps take another
    path; the true residual, recomputed by the oracle in FP64, is what counts
    (cond(D) times rounding is far below the 1e-10 asked for)."""
    from oracle import qed2d as O
    from paper_0811_4331_amd import qed2d
    u = synthetic.u1_gauge_field(dims, 6.0, seed=941)
    m = 0.05
    b = synthetic.gaussian_spinor_2d(dims, seed=942)
    lx, lt = dims
    vecs, n = [], 1
    for k, nv in enumerate(nvs):
        vecs.append(gpu(synthetic.gaussian_vectors((nv, lt, lx, 2, n), 943 + k)))
        lt, lx, n = lt // 4, lx // 4, nv
    c = qed2d.Context2d(dims, "cuda:0")
    c.set_gauge(gpu(u), -1)
    c.set_mass(m)
    c.mg_setup(nvs, vecs, setup_iters=20, coarse_cycles=cycles)
    x, st = c.solve(gpu(b), method="mg-bicgstab", tol=1e-10, maxit=500)
    res = np.linalg.norm(b - O.apply_D(u, x.cpu().numpy(), m, -1.0)) / np.linalg.norm(b)
    assert st["converged"] and res <= 1e-10, (st, res)
    c.close()


@pytest.mark.parametrize("prec,nrhs", [("f16", 5), ("bf16", 8), ("f64", 3)])
def test_prolongation_shared_by_right_hand_sides(prec, nrhs):
    """Batches below the matrix cores' on a lattice large enough for several
    right-hand sides per thread: the same products in the same order as one at
    a time, so equal numbers."""
    ctx, _ = context((16, 16, 16, 16), 951)
    v = synthetic.gaussian_vectors((3, 16, 16, 16, 16, 4, 3), 952)
    ctx.mg_setup([{"block": (4, 4, 4, 4), "nv": 3, "setup_iters": 0, "vectors": gpu(v)}])
    c = synthetic.gaussian_vectors((nrhs,) + tuple(ctx.coarse_shape(1)), 953)
    c = gpu(c if prec == "f64" else c.astype(np.complex64))
    out = ctx.prolong(0, c, prec=prec)
    for j in range(nrhs):
        assert torch.equal(out[j], ctx.prolong(0, c[j].contiguous(), prec=prec)), j
    ctx.close()


@pytest.mark.parametrize("dims", [(8, 8, 8, 16), (4, 4, 8, 8)])  # 1024 and 64 coarse sites
def test_coarsest_solve_of_one_right_hand_side(dims):
    """The coefficients in a launch of their own (many sites) or in the update:
    the cycle's solve to a true residual of 1e-10, recomputed by the oracle."""
    ctx, u = context(dims, 961, -0.3)
    lx, ly, lz, lt = dims
    v = synthetic.gaussian_vectors((4, lt, lz, ly, lx, 4, 3), 962)
    ctx.mg_setup([{"block": (2, 2, 2, 2), "nv": 4, "setup_iters": 20, "vectors": gpu(v)}], coarse_tol=1e-3)
    b = synthetic.gaussian_spinor(dims, seed=963)
    x, st = ctx.solve(gpu(b), tol=1e-10, restart=20, maxit=300)
    st = st[0] if isinstance(st, list) else st
    r = b.reshape(x.shape) - wilson.apply_D(u, x.cpu().numpy(), -0.3, -1.0)
    assert st["converged"] and np.linalg.norm(r) <= 1e-10 * np.linalg.norm(b), st
    ctx.close()


@pytest.mark.parametrize("prec,dims,nrhs", [
    ("f16", (20, 12, 20, 12), 5),     # two right-hand sides per thread, a last group of one; 225 blocks
    ("bf16", (20, 20, 20, 20), 6),    # four per thread, a last group of two; 625 blocks
    ("bf16", (24, 24, 24, 48), 5),    # groups back to back (V longer than 256 MB)
    ("f32", (20, 12, 20, 12), 2),     # the vector units' batch in FP32
])
def test_prolongation_in_groups_of_right_hand_sides(prec, dims, nrhs):
    """Groups of right-hand sides per thread, in either order of the grid, give
    what one at a time gives: the same products in the same order."""
    lx, ly, lz, lt = dims
    ctx = wdmg.Context(dims, DEV)
    u = torch.eye(3, dtype=torch.complex128, device=DEV).expand(ctx.site_shape + (4, 3, 3)).contiguous()
    ctx.set_gauge(u, t_bc=-1)
    ctx.set_mass(0.1)
    g = torch.Generator(device=DEV)
    g.manual_seed(971)
    nv = 12
    v = torch.randn((nv,) + ctx.fine_shape(), generator=g, device=DEV, dtype=torch.complex128)
    ctx.mg_setup([{"block": (4, 4, 4, 4), "nv": nv, "setup_iters": 0, "vectors": v}])
    c = torch.randn((nrhs,) + tuple(ctx.coarse_shape(1)), generator=g, device=DEV, dtype=torch.complex64)
    out = ctx.prolong(0, c, prec=prec)
    for j in range(nrhs):
        assert torch.equal(out[j], ctx.prolong(0, c[j].contiguous(), prec=prec)), j
    ctx.close()
