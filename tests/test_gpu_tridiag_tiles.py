"""Tridiagonal pass along x at the edges of its instances, through the pressure solve by the TPT route.

16 lanes share a line with 2, 4, 5, 6, 7, 8, 10 or 13 rows each (up to 32, 64, 80, 96, 112, 128, 160 and 208
cells), 32 lanes with 8 rows up to 256, 32 and 64 lanes with 16 rows up to 512 and 1024; a wave takes 4, 2 or 1 lines and goes over several
groups of them on large fields.  Lengths on both sides of every limit, line counts that leave a group
partly filled, and enough lines for several groups per wave.  Tolerances of the other instances of the pass:
FP64 1e-11 up to 100 cells and 1e-13 n above, FP32 1e-4 and 2e-6 n_x.
"""
import numpy as np
import pytest

import synth
from oracle import poisson
from oracle.grid import Grid, faces

pytestmark = pytest.mark.gpu

LENGTHS = [2, 3, 15, 16, 17, 31, 32, 33, 64, 65, 80, 81, 96, 97, 112, 113, 128, 129, 160, 161, 208, 209, 255, 256, 257,
           512, 513, 1024]
CASES = [(n, a, b) for n in LENGTHS for a, b in ((2, 2), (3, 5), (7, 9))] + [(5, 97, 101), (33, 95, 97)]


@pytest.mark.parametrize("dims", CASES)
def test_tridiagonal_pass(dims):
    import torch

    import paper_1704_08521_amd as lk
    print(f"[case] {dims}", flush=True)
    fs = [faces(m, "tanh", 10.0) for m in dims]
    g = Grid(*fs)
    c = lk.Context(*dims)
    c.set_grid(*fs)
    r = synth.random_cells(*dims, 400 + sum(dims))
    V = g.volumes()
    r = r - np.sum(V * r) / np.sum(V)
    ref = poisson.PoissonFD(g).solve(r)
    rd = torch.from_numpy(np.ascontiguousarray(r.ravel())).cuda()
    c.set_poisson_method("tpt")
    for prec, bound in ((lk.FP64, max(1e-11, 1e-13 * max(dims))), (lk.MIXED, max(1e-4, 2e-6 * dims[0]))):
        phi = c.poisson_solve(rd, precision=prec).cpu().numpy().reshape(ref.shape)
        err = np.max(np.abs(phi - ref)) / np.max(np.abs(ref))
        assert err < bound, (dims, prec, err)


@pytest.mark.parametrize("n", [40, 230, 300, 600])
def test_lines_do_not_reach_each_other(n):
    # the lines of a wave belong to neighbouring planes y = const of the plane projection: a value that is not
    # finite in one plane leaves the others as they are without it
    import torch

    import paper_1704_08521_amd as lk
    dims = (n, 6, 4)
    print(f"[case] {dims}", flush=True)
    c = lk.Context(*dims)
    c.set_stretching("tanh", 4.0)
    v = synth.random_velocity(*dims, 77)
    bad = v.copy()
    u = bad[:(n + 1) * 6 * 4].reshape(4, 6, n + 1)
    u[2, 3, n // 2] = np.nan
    ref, got = (c.plane_project(torch.from_numpy(f).cuda(), 1)[0].cpu().numpy() for f in (v, bad))
    for off, shape in ((0, (4, 6, n + 1)), ((n + 1) * 24 + n * 28, (5, 6, n))):
        size = int(np.prod(shape))
        a, b = (f[off:off + size].reshape(shape) for f in (ref, got))
        keep = [0, 1, 2, 4, 5]
        assert np.array_equal(a[:, keep], b[:, keep])
    assert np.isnan(got).any()
