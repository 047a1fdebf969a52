"""Momentum stencil at the edges of its tiles against the FP64 oracle.

A block of the kernel covers 60 faces along x and 8 rows along y and a chunk of planes along z:
sizes around those, rows of odd and even length (their last pair of faces is whole or half), and
grids thinner than one tile.  Both forms (Jacobian; residual with the lid) are a fixed, short
sequence of rounded operations per output, hence 1e-12 of the largest value, as for the other
stencil tests.  Wall-normal faces of the input are ignored whatever they hold.
"""
import numpy as np
import pytest

import synth
from oracle import fv
from oracle.grid import Grid

pytestmark = pytest.mark.gpu

DIMS = [(2, 2, 2), (57, 6, 3), (58, 7, 12), (59, 8, 13), (60, 9, 26), (61, 15, 14), (118, 16, 5), (119, 3, 27),
        (120, 17, 2), (121, 2, 40), (5, 23, 70)]


@pytest.mark.parametrize("dims", DIMS)
def test_momentum_tile_edges(dims):
    import torch

    import paper_1704_08521_amd as lk
    print(f"[case] {dims}", flush=True)
    g = Grid.make(*dims, kind="tanh", ratio=10.0)
    c = lk.Context(*dims)
    c.set_stretching("tanh", 10.0)
    c.set_re(900.0)
    c.set_lid(0.4)
    U, v = synth.random_velocity(*dims, 11), synth.random_velocity(*dims, 12)
    walls = g.wall_mask()
    dirty = [np.where(walls, bad, f) for bad, f in ((np.nan, U), (np.inf, v))]
    dev = [torch.from_numpy(f).cuda() for f in dirty]
    c.set_base_flow(torch.from_numpy(U).cuda())
    w = c.jacobian_apply(dev[1]).cpu().numpy()
    r = c.residual(dev[0]).cpu().numpy()
    for got, ref in ((w, fv.jacobian_apply(g, U, v, 900.0)), (r, fv.residual(g, U, 900.0, 0.4))):
        assert np.max(np.abs(got - ref)) <= 1e-12 * np.max(np.abs(ref))
        assert np.all(got[walls] == 0.0)
