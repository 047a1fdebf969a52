"""FP32 left transforms at the edges of their tiles, through the FP32 pressure solve on both routes.

The kernel's variant goes by the line length (a step every 32 points up to 256); a block takes 64 columns
and contracts 16 indices per step.  Lengths on both sides of every limit, odd and even ones, lines of a few
points, on y (segmented columns; on the first route from and to FP64 fields) and on z, with column
counts around one and several blocks.  Tolerance 1e-4, as for the other FP32 instances at short x.
"""
import numpy as np
import pytest

import synth
from oracle import poisson
from oracle.grid import Grid, faces

pytestmark = pytest.mark.gpu

LENGTHS = [2, 3, 7, 8, 9, 31, 32, 33, 40, 64, 65, 96, 97, 128, 129, 160, 161, 192, 193, 224, 225, 255, 256]
OTHERS = [(3, 5), (8, 8), (13, 5), (13, 11)]  # the other two axes: 15, 64, 65 and 143 columns


@pytest.mark.parametrize("axis", [1, 2])
@pytest.mark.parametrize("n", LENGTHS)
def test_left_transform_tiles_fp32(n, axis):
    import torch

    import paper_1704_08521_amd as lk
    for k, (a, b) in enumerate(OTHERS):
        dims = (a, n, b) if axis == 1 else (a, b, n)
        print(f"[case] {dims}", flush=True)
        fs = [faces(m, "tanh", 10.0) for m in dims]
        g = Grid(*fs)
        c = lk.Context(*dims)
        c.set_grid(*fs)
        r = synth.random_cells(*dims, 700 + n + k)
        V = g.volumes()
        r = r - np.sum(V * r) / np.sum(V)
        ref = poisson.PoissonFD(g).solve(r)
        rd = torch.from_numpy(np.ascontiguousarray(r.ravel())).cuda()
        for method in ("tpt", "tpf"):
            c.set_poisson_method(method)
            phi = c.poisson_solve(rd, precision=lk.MIXED).cpu().numpy().reshape(ref.shape)
            err = np.max(np.abs(phi - ref)) / np.max(np.abs(ref))
            assert err < 1e-4, (dims, method, err)
