"""Correction and certificate of a projection pass at the edges of the kernel's tiles.

A block covers 60 faces along x, 8 rows along y and a chunk of planes along z.  One pass of a
projection is compared with the separate entry points: v = w - G p by `correct` from the p it
returned, and the certificate by `divergence` of the v it returned.  Each v is one rounded
product and sum of the same operands, hence 4 eps of the largest term; the certificates are sums of the
same cell values in another order (fewer than 2^20 positive terms), hence 1e-9.
An FP32 pass is far from rounding level, and its D v feeds the second pass, which then gains at least a
factor 100.
"""
import math

import numpy as np
import pytest

import synth
from oracle.grid import Grid

pytestmark = pytest.mark.gpu

DIMS = [(2, 2, 2), (57, 7, 3), (58, 8, 8), (59, 9, 9), (60, 15, 16), (61, 16, 17), (119, 17, 5), (120, 6, 33),
        (121, 2, 70), (5, 23, 2)]


@pytest.mark.parametrize("dims", DIMS)
def test_pass_against_separate_calls(dims):
    import torch

    import paper_1704_08521_amd as lk
    print(f"[case] {dims}", flush=True)
    c = lk.Context(*dims)
    c.set_stretching("tanh", 4.0)
    walls = Grid.make(*dims, kind="tanh", ratio=4.0).wall_mask()
    w = synth.random_velocity(*dims, 21)
    dev = torch.from_numpy(np.where(walls, np.nan, w)).cuda()  # wall-normal faces are not read
    v, p, st = c.project(dev, precision=lk.MIXED, tol=0.0, max_iter=1)
    ref, _ = c.correct(dev, p)
    scale = max(float(ref.abs().max()), float(np.abs(w).max()))
    assert float((v - ref).abs().max()) <= 4 * 2.0**-52 * scale
    assert float(v[torch.from_numpy(walls).cuda()].abs().max()) == 0.0
    _, n0 = c.divergence(torch.from_numpy(w).cuda())
    _, n1 = c.divergence(v)
    assert math.isclose(st["rho"], n1 / n0, rel_tol=1e-9)
    _, _, st2 = c.project(dev, precision=lk.MIXED, tol=0.0, max_iter=2)
    assert st2["rho"] <= max(1e-2 * st["rho"], 1e-12)
