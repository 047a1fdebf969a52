"""Gram-Schmidt passes at the edges of their tiles, through the Arnoldi driver.

The dot products take eight vectors per block and 32 per launch, the norm of the new vector beside them as one
more; values are read in pairs, so vectors of odd length end in half a pair.  Up to 48 vectors the first update
leaves the dot products of a second pass.  Basis sizes on both sides of 8, 16, 32, 40 and 48 vectors,
velocities of even and odd length.  The Ritz pairs are checked with the oracle's own
operator: residuals of 1e-8 for a tolerance of 1e-10, as the driver's estimate holds up to the loss of
orthogonality that a wrong projection coefficient would cause.
"""
import pytest

from oracle import eigen
from oracle.grid import Grid
from oracle.newton import Newton

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [15, 16, 17, 31, 32, 33, 41, 50])
@pytest.mark.parametrize("dims", [(8, 8, 8), (8, 7, 7)])
def test_ritz_pairs_by_basis_size(dims, m):
    import torch

    import paper_1704_08521_amd as lk
    print(f"[case] {dims} m = {m}", flush=True)
    g = Grid.make(*dims)
    U, _ = Newton(g, 60.0, 0.0).solve(tol=1e-12)
    c = lk.Context(*dims)
    c.set_stretching("uniform")
    c.set_re(60.0)
    c.set_base_flow(torch.from_numpy(U).cuda())
    out = c.arnoldi_leading(k=3, m=m, tol=1e-10, max_restarts=400, seed=2, vectors=True)
    assert out["converged"]
    vre, vim = out["vectors"]
    for q in range(len(out["eig"])):
        x = vre[q].cpu().numpy() + 1j * vim[q].cpu().numpy()
        assert eigen.ritz_residual(g, U, 60.0, out["eig"][q], x) < 1e-8
