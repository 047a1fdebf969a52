"""FP64 left transforms of more than 10000 columns, through the pressure solve on both routes.

Lines of more than 120 points go by the number of columns too: up to 10000 one variant serves every length,
beyond it there is one each up to n = 128, 160, 176, 208 and 256.  Lengths on both sides of these limits, odd and even
ones, with 9999, 10000 and 10100 columns on y (segmented) and on z.  Tolerance as for the other transform
instances, 1e-13 n.
"""
import numpy as np
import pytest

import synth
from oracle import poisson
from oracle.grid import Grid, faces

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("axis", [1, 2])
@pytest.mark.parametrize("n", [120, 121, 127, 128, 129, 159, 160, 161, 176, 177, 207, 208, 209, 255, 256])
def test_left_transforms_of_many_columns(n, axis):
    import torch

    import paper_1704_08521_amd as lk
    for a, b in [(101, 100)] + ([(101, 99), (100, 100)] if n in (121, 208) else []):
        dims = (a, n, b) if axis == 1 else (a, b, n)
        print(f"[case] {dims}", flush=True)
        fs = [faces(m, "tanh", 10.0) for m in dims]
        g = Grid(*fs)
        c = lk.Context(*dims)
        c.set_grid(*fs)
        r = synth.random_cells(*dims, 300 + n)
        V = g.volumes()
        r = r - np.sum(V * r) / np.sum(V)
        ref = poisson.PoissonFD(g).solve(r)
        rd = torch.from_numpy(np.ascontiguousarray(r.ravel())).cuda()
        for method in ("tpt", "tpf"):
            c.set_poisson_method(method)
            phi = c.poisson_solve(rd).cpu().numpy().reshape(ref.shape)
            err = np.max(np.abs(phi - ref)) / np.max(np.abs(ref))
            assert err < 1e-13 * n, (dims, method, err)
