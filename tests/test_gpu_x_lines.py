"""FP64 transforms along x at the edges of their tiles, through the pressure solve by the TPF route.

Lines are taken as columns whose rows are neighbours: lengths on both sides of the limits of the kernel's
variants (groups of eight points up to n = 64, 120, 160 and 208 with mirror symmetry, then the kernel for
lines; 136, 208 and 256 without), odd and even ones, with line counts around one and several tiles of 16.
Tolerance as for the other transform instances.
"""
import numpy as np
import pytest

import synth
from oracle import poisson
from oracle.grid import Grid, faces

pytestmark = pytest.mark.gpu

LENGTHS = [2, 3, 4, 5, 7, 8, 9, 63, 65, 119, 121, 136, 137, 160, 161, 207, 208, 209, 225, 256, 257]
OTHERS = [(3, 5), (4, 4), (11, 3), (13, 11)]  # 15, 16, 33 and 143 lines


def skewed(n):
    d = np.linspace(1.0, 2.0, n) ** 1.5
    f = np.concatenate([[0.0], np.cumsum(d) / np.sum(d)])
    f[-1] = 1.0
    return f


@pytest.mark.parametrize("symmetric", [True, False])
@pytest.mark.parametrize("n", LENGTHS)
def test_transforms_along_x(n, symmetric):
    import torch

    import paper_1704_08521_amd as lk
    for k, (a, b) in enumerate(OTHERS):
        dims = (n, a, b)
        print(f"[case] {dims} symmetric = {symmetric}", flush=True)
        fs = [faces(m, "tanh", 10.0) if symmetric or q else skewed(m) for q, m in enumerate(dims)]
        g = Grid(*fs)
        c = lk.Context(*dims)
        c.set_grid(*fs)
        r = synth.random_cells(*dims, 500 + n + k)
        V = g.volumes()
        r = r - np.sum(V * r) / np.sum(V)
        ref = poisson.PoissonFD(g).solve(r)
        c.set_poisson_method("tpf")
        phi = c.poisson_solve(torch.from_numpy(np.ascontiguousarray(r.ravel())).cuda()).cpu().numpy().reshape(ref.shape)
        err = np.max(np.abs(phi - ref)) / np.max(np.abs(ref))
        assert err < max(1e-11, 1e-13 * n), (dims, symmetric, err)
