"""FP64 transforms along x on both sides of every limit of the rule that gives mirror-symmetric axes to the left
kernels or to those for lines (multiples of 16 from 96 on, 161 to 192 points and more than 208 go to the latter),
through the pressure solve by the TPF route and through the viscous step, whose face axis has one point more.
Tolerances as for the other instances of each: 1e-11 up to 100 points and 1e-13 n above, 1e-11 for the
viscous step.
"""
import numpy as np
import pytest

import synth
from oracle import poisson, stokes
from oracle.grid import Grid, faces

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [79, 80, 81, 95, 96, 97, 111, 112, 128, 143, 144, 159, 160, 161, 175, 176, 191, 192, 193,
                               207, 208, 209])
def test_transforms_along_x_by_rule(n):
    import torch

    import paper_1704_08521_amd as lk
    for a, b in [(3, 5), (13, 11)]:
        dims = (n, a, b)
        print(f"[case] {dims}", flush=True)
        fs = [faces(m, "tanh", 10.0) for m in dims]
        g = Grid(*fs)
        c = lk.Context(*dims)
        c.set_grid(*fs)
        c.set_re(50.0)
        r = synth.random_cells(*dims, 800 + n)
        V = g.volumes()
        r = r - np.sum(V * r) / np.sum(V)
        ref = poisson.PoissonFD(g).solve(r)
        c.set_poisson_method("tpf")
        phi = c.poisson_solve(torch.from_numpy(np.ascontiguousarray(r.ravel())).cuda()).cpu().numpy().reshape(ref.shape)
        assert np.max(np.abs(phi - ref)) < max(1e-11, 1e-13 * n) * np.max(np.abs(ref)), dims
        if a == 3:
            f = synth.random_velocity(*dims, 900 + n)
            u = c.viscous_solve(torch.from_numpy(f).cuda(), 0.1).cpu().numpy()
            ref = stokes.viscous_solve(g, f, 50.0, 0.1)
            assert np.max(np.abs(u - ref)) < 1e-11 * np.max(np.abs(ref)), dims
