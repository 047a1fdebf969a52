"""Tridiagonal pass along x: lanes per line by the number of lines, and the accuracy of its FP32 solves.

Up to 1600 lines (20000 past 256 cells) a line has all 64 lanes, with 2, 4 or 8 rows each up to 128, 256 and 512 cells;
beyond it 16 or 32 lanes.  Lengths on both sides of these limits with line counts on both sides.  FP64: 1e-11 up
to 100 cells and 1e-13 n above.

FP32: the elimination has no subtraction, so a solve is as good as its rounded factors and sums: each of the
two transforms is an inner product of up to n rounded terms, whose errors add up like sqrt(n) eps, and the
rows of a line likewise, 4 sqrt(n) eps in all with eps = 2^-23: 2e-6 at 16, 1e-5 at 400, 1.5e-5 at 1024.  An elimination
that forms its pivots by differences misses that by one to two orders of magnitude.
"""
import numpy as np
import pytest

import synth
from oracle import poisson
from oracle.grid import Grid, faces

pytestmark = pytest.mark.gpu

CASES = [(n, a, b) for n in (64, 65, 127, 128, 129, 255, 256) for a, b in ((3, 5), (40, 40), (39, 43))]
CASES += [(n, a, b) for n in (257, 511, 512, 513) for a, b in ((2, 2), (3, 5))]
CASES += [(257, 125, 160), (257, 143, 140)]


def problem(dims, ratio=10.0):
    import torch

    import paper_1704_08521_amd as lk
    print(f"[case] {dims}", flush=True)
    fs = [faces(m, "tanh", ratio) for m in dims]
    g = Grid(*fs)
    c = lk.Context(*dims)
    c.set_grid(*fs)
    r = synth.random_cells(*dims, 600 + sum(dims))
    V = g.volumes()
    r = r - np.sum(V * r) / np.sum(V)
    return lk, c, torch.from_numpy(np.ascontiguousarray(r.ravel())).cuda(), poisson.PoissonFD(g).solve(r)


def error(c, rd, ref, prec):
    phi = c.poisson_solve(rd, precision=prec).cpu().numpy().reshape(ref.shape)
    return np.max(np.abs(phi - ref)) / np.max(np.abs(ref))


@pytest.mark.parametrize("dims", CASES)
def test_lanes_by_lines(dims):
    lk, c, rd, ref = problem(dims)
    assert error(c, rd, ref, lk.FP64) < max(1e-11, 1e-13 * max(dims))
    assert error(c, rd, ref, lk.MIXED) < 4 * np.sqrt(max(dims)) * 2.0**-23


@pytest.mark.parametrize("dims", [(2, 3, 5), (16, 7, 9), (33, 8, 8), (64, 5, 6), (100, 40, 41), (208, 6, 7), (209, 50, 40),
                                  (400, 4, 5), (600, 3, 3), (1024, 2, 3)])
def test_fp32_solve_accuracy(dims):
    lk, c, rd, ref = problem(dims)
    assert error(c, rd, ref, lk.MIXED) < 4 * np.sqrt(max(dims)) * 2.0**-23
