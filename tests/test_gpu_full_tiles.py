"""FP64 left transforms of axes without mirror symmetry at the edges of their tiles, through the pressure solve.

The full matrix is contracted with its lower rows (he = ceil(n/2)) and its upper rows side by side, in row
groups of four; the variant goes by the number of groups of a half (up to 17, 26 and 32: n = 136,
208, 256; longer axes take the vector units).  Lengths on both sides of every limit, odd and even ones and
lines of a few points, on y (segmented columns) and on z (with the eigenvalue division on the second
route), next to axes with and without the symmetry.  Tolerance as for the other transform instances.
"""
import numpy as np
import pytest

import synth
from oracle import poisson
from oracle.grid import Grid, faces

pytestmark = pytest.mark.gpu

LENGTHS = [3, 4, 5, 7, 8, 9, 31, 33, 65, 121, 135, 136, 137, 207, 208, 209, 255, 256, 257]
OTHERS = [(3, 5), (4, 4), (11, 3), (13, 11)]  # the other two axes: 15, 16, 33 and 143 columns


def skewed(n):
    d = np.linspace(1.0, 2.0, n) ** 1.5
    f = np.concatenate([[0.0], np.cumsum(d) / np.sum(d)])
    f[-1] = 1.0
    return f


@pytest.mark.parametrize("axis", [1, 2])
@pytest.mark.parametrize("n", LENGTHS)
def test_full_left_transform_tiles(n, axis):
    import torch

    import paper_1704_08521_amd as lk
    for k, (a, b) in enumerate(OTHERS):
        dims = (a, n, b) if axis == 1 else (a, b, n)
        print(f"[case] {dims}", flush=True)
        fs = [skewed(m) if q == axis or k % 2 else faces(m, "tanh", 10.0) for q, m in enumerate(dims)]
        g = Grid(*fs)
        c = lk.Context(*dims)
        c.set_grid(*fs)
        r = synth.random_cells(*dims, 300 + n + k)
        V = g.volumes()
        r = r - np.sum(V * r) / np.sum(V)
        ref = poisson.PoissonFD(g).solve(r)
        rd = torch.from_numpy(np.ascontiguousarray(r.ravel())).cuda()
        for method in ("tpt", "tpf"):
            c.set_poisson_method(method)
            phi = c.poisson_solve(rd).cpu().numpy().reshape(ref.shape)
            err = np.max(np.abs(phi - ref)) / np.max(np.abs(ref))
            assert err < max(1e-11, 1e-13 * n), (dims, method, err)
