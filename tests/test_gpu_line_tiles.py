"""FP64 left transforms at the edges of their tiles, through the pressure solve on both routes.

The kernel's variant goes by the number of groups of eight points of the line (up to 8, 15, 20, 26 and 32
groups: n = 64, 120, 160, 208, 256), each variant splitting the groups into classes; a wave takes 16 or 32
columns.  Lengths on both sides of every limit, odd and even ones, lines of a few points, on y
(segmented columns) and on z, with column counts around one and several waves.  Tolerance: an n-term
inner product of rounded factors per transform on both sides, 1e-11 up to n = 100 and 1e-13 n above, as for the
other transform instances.
"""
import numpy as np
import pytest

import synth
from oracle import poisson
from oracle.grid import Grid, faces

pytestmark = pytest.mark.gpu

LENGTHS = [2, 3, 4, 5, 7, 8, 9, 63, 64, 65, 119, 120, 121, 160, 161, 208, 209, 255, 256]
OTHERS = [(3, 5), (4, 4), (11, 3), (13, 11)]  # the other two axes: 15, 16, 33 and 143 columns


@pytest.mark.parametrize("axis", [1, 2])
@pytest.mark.parametrize("n", LENGTHS)
def test_left_transform_tiles(n, axis):
    import torch

    import paper_1704_08521_amd as lk
    for k, (a, b) in enumerate(OTHERS):
        dims = (a, n, b) if axis == 1 else (a, b, n)
        print(f"[case] {dims}", flush=True)
        fs = [faces(m, "tanh", 10.0) for m in dims]
        g = Grid(*fs)
        c = lk.Context(*dims)
        c.set_grid(*fs)
        r = synth.random_cells(*dims, 900 + n + k)
        V = g.volumes()
        r = r - np.sum(V * r) / np.sum(V)
        ref = poisson.PoissonFD(g).solve(r)
        rd = torch.from_numpy(np.ascontiguousarray(r.ravel())).cuda()
        for method in ("tpt", "tpf"):
            c.set_poisson_method(method)
            phi = c.poisson_solve(rd).cpu().numpy().reshape(ref.shape)
            err = np.max(np.abs(phi - ref)) / np.max(np.abs(ref))
            assert err < max(1e-11, 1e-13 * n), (dims, method, err)
