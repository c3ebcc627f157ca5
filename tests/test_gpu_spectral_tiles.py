"""Fourier-differentiation operator at the edges of its launch: 16 x 16 and 32 x 32 tiles, ragged rows,
columns and k ranges, against the oracle."""
import numpy as np
import pytest

from synth import rng_for, uniform_velocity

# (nx, ny, npml): one tile with a partial one beside it, k ranges of 1 and 7 past whole chunks, and a
# grid of 256 ragged 32 x 32 tiles (the large tile's smallest launch) that is not square
GRIDS = [(13, 3, 2), (12, 21, 2), (477, 483, 2)]


@pytest.mark.gpu
@pytest.mark.parametrize("nx,ny,npml", GRIDS)
@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("dtype,tol", [("complex64", 1e-5), ("complex128", 1e-12)])
def test_apply_matches_oracle(nx, ny, npml, adjoint, dtype, tol):
    import torch
    from oracle import helmholtz as ohz
    from oracle import spectral as osp
    from paper_2607_16906_amd import hz
    from synth import C_REF, H_10PPW
    nxt, nyt = nx + 2 * npml, ny + 2 * npml
    rng = rng_for(78, 1, nxt)
    c = np.abs(uniform_velocity(max(nxt, nyt), rng)[:nyt, :nxt]).astype(np.float32)
    u = (rng.standard_normal((nyt, nxt)) + 1j * rng.standard_normal((nyt, nxt))).astype(dtype)
    op = ohz.Problem(c.astype(np.float64), npml, H_10PPW, 1.0, 2.0, C_REF)
    gp = hz.Problem(c.ravel(), nx, ny, npml, H_10PPW, 1.0, 2.0, C_REF, disc="spectral")
    got = gp.apply(torch.from_numpy(u.ravel()).cuda(), adjoint=adjoint).cpu().numpy().reshape(nyt, nxt)
    ref = (osp.op_adjoint if adjoint else osp.op_apply)(op, u.astype(np.complex128))
    assert np.linalg.norm(got - ref) <= tol * np.linalg.norm(ref)
