"""Fourier-differentiation operator: the real and the imaginary part each as accurate as the other, however
unlike their sizes, and the residual forms on a grid of 32 x 32 tiles."""
import numpy as np
import pytest

from synth import rng_for


def build(nx, ny, npml, seed):
    from oracle import helmholtz as ohz
    from paper_2607_16906_amd import hz
    from synth import C_REF, H_10PPW
    nxt, nyt = nx + 2 * npml, ny + 2 * npml
    c = rng_for(101, 1, seed).uniform(1400.0, 2800.0, (nyt, nxt)).astype(np.float32)
    op = ohz.Problem(c.astype(np.float64), npml, H_10PPW, 1.0, 2.0, C_REF)
    return op, hz.Problem(c.ravel(), nx, ny, npml, H_10PPW, 1.0, 2.0, C_REF, disc="spectral")


@pytest.mark.gpu
@pytest.mark.parametrize("nx,ny", [(61, 46), (296, 296), (481, 487)])   # 16 x 16 tiles, the same in rounds, 32 x 32
@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("dtype,tol", [("complex64", 5e-6), ("complex128", 1e-12)])
@pytest.mark.parametrize("small", ["re", "im"])
def test_small_part_keeps_its_accuracy(nx, ny, adjoint, dtype, tol, small):
    # without absorbing layers A is real: the part of size 1e-6 is A times that part of the field, and its error
    # does not depend on the large one. Sums of up to 487 products: 2^-24 sqrt(487) = 1.3e-6 of the terms' norm;
    # the matrices' own rounding in FP64
    import torch
    from oracle import spectral as osp
    op, gp = build(nx, ny, 0, nx)
    g = rng_for(101, 2, nx)
    re, im = (g.standard_normal((ny, nx)).astype(dtype).real for _ in range(2))
    re, im = (re * 1e-6, im) if small == "re" else (re, im * 1e-6)
    u = (re + 1j * im).astype(dtype)
    got = gp.apply(torch.from_numpy(u.ravel()).cuda(), adjoint=adjoint).cpu().numpy().reshape(ny, nx)
    f = osp.op_adjoint if adjoint else osp.op_apply
    for part in ("real", "imag"):
        ref = f(op, getattr(u, part).astype(np.complex128)).real
        assert np.linalg.norm(getattr(got, part) - ref) <= tol * np.linalg.norm(ref), part


@pytest.mark.gpu
def test_residual_fp64_large_tiles():
    # the solver's FP64 residual at a grid of 256 ragged 32 x 32 tiles
    import torch
    from oracle import spectral as osp
    from paper_2607_16906_amd import hz
    op, gp = build(477, 483, 2, 3)
    g = rng_for(101, 3, 0)
    b = g.standard_normal((487, 481)) + 1j * g.standard_normal((487, 481))
    x, info = hz.fgmres(gp, torch.from_numpy(b.ravel()).cuda(), m=3, tol=1e-12, maxit=3, krylov="c128")
    r = b - osp.op_apply(op, x.cpu().numpy().reshape(487, 481))
    rel = np.linalg.norm(r) / np.linalg.norm(b)
    assert 0 < rel < 1 and abs(info.true_relres - rel) <= 1e-12


@pytest.mark.gpu
def test_residual_fp32_large_tiles():
    # the training loss's FP32 residual at the same grid
    import torch
    from oracle import spectral as osp, unet
    from paper_2607_16906_amd import hz
    from synth import he_uniform
    op, gp = build(477, 483, 2, 4)
    g = rng_for(101, 4, 0)
    r = (g.standard_normal((1, 487, 481)) + 1j * g.standard_normal((1, 487, 481))).astype(np.complex64)
    specs = unet.layer_specs(1, 8, 5)
    theta = he_uniform(unet.init_shapes(specs), rng_for(101, 5, 0))
    net = hz.Net(1, 8, 5, theta)
    loss, per, _ = hz.loss_backward(net, [gp], torch.from_numpy(r.reshape(1, -1)).cuda(), prec="fp32", need_grad=False)
    ref, _, _ = unet.loss_and_grad(theta.astype(np.float64), specs, [op], r.astype(np.complex128), need_grad=False,
                                   ops=osp)
    assert abs(float(loss) - ref) <= 1e-5 * ref and abs(float(per[0]) - ref) <= 1e-5 * ref
