"""What a projection leaves in the caller's outputs when its input ends it early.

A momentum update whose divergence is not finite is refused before anything of the caller's is written, in
every form and on both routes of the solve; one with no divergence at all is returned as it is
(p = 0, no pass).  Both are decided from the sum of V (D w)^2, whose terms the host adds on small grids and the
device on large ones: (16, 14, 12) has 16 of them, (4, 256, 100) 1600.
"""
import numpy as np
import pytest

import synth
from oracle.grid import Grid

pytestmark = pytest.mark.gpu

DIMS = [(16, 14, 12), (4, 256, 100)]


def context(dims, route):
    import paper_1704_08521_amd as lk
    c = lk.Context(*dims)
    c.set_stretching("tanh", 4.0)
    c.set_poisson_method(route)
    return lk, c


@pytest.mark.parametrize("route", ["tpt", "tpf"])
@pytest.mark.parametrize("dims", DIMS)
def test_refused_input_leaves_the_outputs(dims, route):
    import torch
    print(f"[case] {dims} {route}", flush=True)
    lk, c = context(dims, route)
    net = lk.Net(3)
    c.set_net(net)
    w = synth.random_velocity(*dims, 5)
    inside = np.flatnonzero(~Grid.make(*dims, kind="tanh", ratio=4.0).wall_mask())
    good = torch.from_numpy(w).cuda()
    first = c.project(good, tol=1e-10)
    for bad in (np.nan, np.inf, 1e200):  # (the square of the last one's divergence overflows)
        f = w.copy()
        f[inside[len(inside) // 3]] = bad
        dev = torch.from_numpy(f).cuda()
        for form in (lk.FP64, lk.MIXED, lk.LEARNED):
            v, p = torch.full_like(c.vel(), 7.5), torch.full_like(c.cells(), -2.5)
            with pytest.raises(lk.LidKrylovError) as e:
                c.project(dev, v, p, precision=form, tol=1e-10)
            assert e.value.code == lk._lib.LC_EINVAL
            assert bool((v == 7.5).all()) and bool((p == -2.5).all()), (bad, form)
    # and the context is as it was
    again = c.project(good, tol=1e-10)
    assert torch.equal(first[0], again[0]) and torch.equal(first[1], again[1])


@pytest.mark.parametrize("route", ["tpt", "tpf"])
@pytest.mark.parametrize("dims", DIMS)
def test_input_without_divergence(dims, route):
    import torch
    print(f"[case] {dims} {route}", flush=True)
    lk, c = context(dims, route)
    # entries whose squared divergence underflows: the norm is zero, and the input the answer
    w = 1e-170 * synth.random_velocity(*dims, 6)
    walls = Grid.make(*dims, kind="tanh", ratio=4.0).wall_mask()
    ref = torch.from_numpy(np.where(walls, 0.0, w)).cuda()
    dev = torch.from_numpy(np.where(walls, 3.0, w)).cuda()
    for form in (lk.FP64, lk.MIXED):
        v, p = torch.full_like(c.vel(), 7.5), torch.full_like(c.cells(), -2.5)
        _, _, st = c.project(dev, v, p, precision=form, tol=1e-10)
        assert st["iterations"] == 0 and st["rho0"] == 0.0 and st["converged"]
        assert torch.equal(v, ref) and not p.any()
