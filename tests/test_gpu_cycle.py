"""One restart cycle without a preconditioner: at the lengths where the update kernels and the triangular
solve change form, on grids around a block's 256 points, the residual of x is the cycle's estimate."""
import pytest

from synth import H_10PPW, rng_for


@pytest.mark.gpu
@pytest.mark.parametrize("krylov,tol", [("c64", 1e-4), ("c128", 1e-10)])
@pytest.mark.parametrize("nx,ny", [(8, 8), (9, 21), (60, 52), (33, 71)])   # 256 points, odd counts, a part block
@pytest.mark.parametrize("m", [1, 8, 9, 24, 25, 32, 33, 48, 49, 64])
def test_estimate_is_the_residual(m, nx, ny, krylov, tol):
    # the estimate follows the Givens rotations alone; it equals ||b - A x|| / ||b|| as long as the basis is
    # orthonormal and y solves the triangle: up to m roundings of vectors of norm about 1 (2^-24 or 2^-53
    # each), which |y| and |A| of order 10 may enlarge
    import torch
    from paper_2607_16906_amd import hz
    n = (nx + 8) * (ny + 8)
    gp = hz.Problem(rng_for(97, 1, n).uniform(1400.0, 2800.0, n), nx, ny, 4, H_10PPW)
    g = rng_for(97, 2, n)
    b = torch.from_numpy(g.standard_normal(n) + 1j * g.standard_normal(n)).cuda()
    x, info = hz.fgmres(gp, b, m=m, tol=1e-14, maxit=m, krylov=krylov)
    res = float((b - gp.apply(x)).norm() / b.norm())
    assert info.its == m and 0 < res < 1
    assert abs(res - float(info.hist[m - 1])) <= tol
