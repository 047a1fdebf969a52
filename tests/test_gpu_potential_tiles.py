"""Vector potentials of the plane projections at the edges of the scans' tiles.

A wave scans a row 64 values at a time, four such pieces loaded together (n = 64, 128, 256); a column is
scanned in eight segments kept in registers up to 8, 20 or 32 rows each (n = 64, 160, 256) and read
twice beyond.  Each potential is the prefix sum of the returned field: n terms summed in some order on either side,
hence n eps times the sum of their absolute values.
"""
import numpy as np
import pytest

import synth
from oracle.grid import Grid

pytestmark = pytest.mark.gpu

LENGTHS = [2, 7, 8, 9, 63, 64, 65, 127, 129, 160, 161, 255, 256, 257, 300]


@pytest.mark.parametrize("which", [1, 2, 3])
@pytest.mark.parametrize("n", LENGTHS)
def test_potential_is_the_prefix_sum(n, which):
    import torch

    import paper_1704_08521_amd as lk
    dims = (5, n, 3) if which == 2 else (n, 5, 3)
    print(f"[case] {dims} P{which}", flush=True)
    nx, ny, nz = dims
    g = Grid.make(*dims, kind="tanh", ratio=4.0)
    c = lk.Context(*dims)
    c.set_stretching("tanh", 4.0)
    v = torch.from_numpy(synth.random_velocity(*dims, 31 + n)).cuda()
    out, psi = c.plane_project(v, which)
    out, psi = out.cpu().numpy(), psi.cpu().numpy()
    nu, nv = (nx + 1) * ny * nz, nx * (ny + 1) * nz
    if which == 3:
        f, d, ax, sgn = out[nu:nu + nv].reshape(nz, ny + 1, nx), g.X.d, 2, -1.0
    else:
        f = out[nu + nv:].reshape(nz + 1, ny, nx)
        d, ax, sgn = (g.X.d, 2, 1.0) if which == 1 else (g.Y.d, 1, -1.0)
    t = sgn * f * (d if ax == 2 else d[:, None])
    pad = [(0, 0)] * 3
    pad[ax] = (1, 0)
    ref = np.pad(np.cumsum(t, axis=ax), pad)
    bound = n * 2.0**-52 * np.sum(np.abs(t), axis=ax, keepdims=True)
    assert np.all(np.abs(psi.reshape(ref.shape) - ref) <= bound)
