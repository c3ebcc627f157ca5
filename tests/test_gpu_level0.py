"""Level 0 of the BF16 network as two launches against one launch per layer, at padded grids around the
launches' 14 x 14 output tiles, and the batch against its systems."""
import numpy as np
import pytest

from synth import H_10PPW, he_uniform, rng_for

# interior sizes whose padded grids (with 4 absorbing layers on each side, rounded up to a multiple of 4) are one tile and
# less, one column more than a tile, several tiles and a remainder, and rows unlike columns
SIZES = [(5, 1), (6, 6), (8, 17), (20, 7), (39, 24), (3, 70)]


def build(sizes):
    import torch
    from paper_2607_16906_amd import hz
    theta = he_uniform(hz.init_shapes(3, 32, 5), rng_for(83, 1, 0))
    net = hz.Net(3, 32, 5, theta)
    gps, vs = [], []
    for i, (nx, ny) in enumerate(sizes):
        c = rng_for(83, 2, i).uniform(1400.0, 2800.0, (ny + 8) * (nx + 8))
        gp = hz.Problem(c, nx, ny, 4, H_10PPW)
        g = rng_for(83, 3, i)
        gps.append(gp)
        vs.append(torch.from_numpy(g.standard_normal(gp.n) + 1j * g.standard_normal(gp.n)).cuda())
    return net, gps, vs


@pytest.mark.gpu
@pytest.mark.parametrize("size", SIZES)
@pytest.mark.parametrize("dtype", ["complex64", "complex128"])
def test_same_bits_as_separate_layers(size, dtype):
    import torch
    net, (gp,), (v,) = build([size])
    v = v.to(getattr(torch, dtype))
    outs = []
    for mode in (2, 0, 1):
        net.set_fused_upsampling(mode)
        outs.append(net.apply(gp, v, prec="bf16"))
    assert float(outs[0].abs().max()) > 0
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])


@pytest.mark.gpu
@pytest.mark.parametrize("mode", [0, 2])
def test_batch_equals_single(mode):
    # one preconditioned step of each system: no restart, so the iterate is that of its own solve up to
    # the contraction choices of the batched Krylov kernels (FP32 basis: 1e-5)
    import torch
    from paper_2607_16906_amd import hz
    net, gps, vs = build(SIZES)
    net.set_fused_upsampling(mode)
    bs = [v.to(torch.complex64) for v in vs]
    xs, _ = hz.fgmres_batched(gps, bs, net=net, m=4, tol=1e-12, maxit=1, krylov="c64", net_prec="bf16")
    for gp, b, x in zip(gps, bs, xs):
        ref, _ = hz.fgmres(gp, b, net=net, m=4, tol=1e-12, maxit=1, krylov="c64", net_prec="bf16")
        assert float((x - ref).norm()) <= 1e-5 * float(ref.norm())
