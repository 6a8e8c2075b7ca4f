"""One right-hand side in 16 bits, which fetches both neighbours' rows at once,
against the same field as both members of a batch: the operator to the rounding
of its result, and MR steps, whose sums it leaves too."""
import numpy as np
import pytest
import torch

import synthetic
from oracle import precision
from paper_0811_4331_amd import wdmg

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("prec", ["f16", "bf16"])
@pytest.mark.parametrize("dims", [(8, 8, 8, 8),    # whole tiles
                                  (6, 4, 2, 10),   # 480 sites: the last block half empty
                                  (3, 5, 3, 7),    # odd extents
                                  (2, 2, 2, 2)])   # 16 sites, neighbours of each other both ways
def test_one_right_hand_side(dims, prec):
    ctx = wdmg.Context(dims, DEV)
    ctx.set_gauge(torch.from_numpy(synthetic.gauge_field(dims, 0.35, 1011)).to(DEV), t_bc=-1)
    ctx.set_mass(-0.4)
    ctx.set_tuning("dslash", 1)
    ctx.set_tuning("dslash_group", 2)
    f = synthetic.gaussian_spinor(dims, seed=1012, nrhs=1).astype(np.complex64)
    f = torch.from_numpy(f).to(DEV).reshape(ctx.fine_shape())
    two = torch.stack([f, f])
    one, pair = ctx.apply_D(f, prec=prec), ctx.apply_D(two, prec=prec)
    assert torch.equal(pair[0], pair[1])
    top = torch.view_as_real(pair[0]).abs().amax(dim=(-3, -2, -1), keepdim=True)
    # a rounding of the FP32 result may fall either way: one unit of the site's scale
    assert bool((torch.view_as_real(one - pair[0]).abs() <= (2 * precision.HALF_ULP[prec] + 1e-6) * top).all())
    x1 = ctx.smooth(0, torch.zeros_like(f), f, 4, prec=prec)
    x2 = ctx.smooth(0, torch.zeros_like(two), two, 4, prec=prec)[0]
    # four steps, each of which may round a unit either way in x and in r
    assert float((x1 - x2).abs().max() / x2.abs().max()) <= 16 * precision.HALF_ULP[prec]
    ctx.close()


@pytest.mark.parametrize("prec", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("group", [1, 2, 3, 7, 64])
def test_groups_of_right_hand_sides(prec, group):
    """Seven right-hand sides in groups of one, two, three, all, and more than
    there are, on a lattice whose last block of 64 sites is half empty.  A group
    works on each of its right-hand sides alone, with the same operations: equal
    numbers, but for one in 16 bits, which has a kernel of its own."""
    dims, nrhs = (6, 4, 2, 10), 7
    ctx = wdmg.Context(dims, DEV)
    ctx.set_gauge(torch.from_numpy(synthetic.gauge_field(dims, 0.35, 1021)).to(DEV), t_bc=-1)
    ctx.set_mass(-0.4)
    ctx.set_tuning("dslash", 1)
    f = synthetic.gaussian_spinor(dims, seed=1022, nrhs=nrhs)
    f = torch.from_numpy(f if prec == "f64" else f.astype(np.complex64)).to(DEV)
    ctx.set_tuning("dslash_group", 5)
    want, wx = ctx.apply_D(f, prec=prec), ctx.smooth(0, torch.zeros_like(f), f, 3, prec=prec)
    ctx.set_tuning("dslash_group", group)
    got, gx = ctx.apply_D(f, prec=prec), ctx.smooth(0, torch.zeros_like(f), f, 3, prec=prec)
    if group == 1 and prec in ("f16", "bf16"):
        top = torch.view_as_real(want).abs().amax(dim=(-3, -2, -1), keepdim=True)
        assert bool((torch.view_as_real(got - want).abs() <= (2 * precision.HALF_ULP[prec] + 1e-6) * top).all())
    else:
        assert torch.equal(got, want) and torch.equal(gx, wx)
    ctx.close()
