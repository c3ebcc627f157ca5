"""Weight gradients at grids around the kernels' tiles: a batch against its samples, and against a plain
statement of the network differentiated in float64."""
import numpy as np
import pytest

from synth import H_10PPW, he_uniform, rng_for

# padded sizes: 8 and 16 columns and one group more, heights below, at and across the tiles of 16 and
# 32 rows (a batch's rows run through them with a row of zeros between the samples)
GRIDS = [(8, 8), (16, 12), (20, 36), (24, 16), (36, 20), (68, 40)]


def build(levels, base, W, H, B):
    import torch
    from paper_2607_16906_amd import hz
    theta = he_uniform(hz.init_shapes(levels, base, 5), rng_for(89, 1, base))
    net = hz.Net(levels, base, 5, theta)
    gps = [hz.Problem(rng_for(89, 2, b).uniform(1400.0, 2800.0, H * W), W - 4, H - 4, 2, H_10PPW) for b in range(B)]
    g = rng_for(89, 3, W)
    r = torch.from_numpy(g.standard_normal((B, H * W)) + 1j * g.standard_normal((B, H * W)))
    return net, theta, gps, r.to(torch.complex64).cuda()


def per_layer(levels, base, grad):
    from paper_2607_16906_amd import hz
    out, off = [], 0
    for s, nb, _ in hz.init_shapes(levels, base, 5):
        for k in (int(np.prod(s)), nb):
            out.append(grad[off:off + k].double())
            off += k
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["bf16", "fp32"])
@pytest.mark.parametrize("W,H", GRIDS)
@pytest.mark.parametrize("levels,base", [(3, 8), (3, 32)])   # 16 to 128 channels as stored
def test_batch_is_the_mean_of_its_samples(levels, base, W, H, prec):
    # a sample's activations do not depend on its batch and its activation gradients only by the exact
    # factor 1 / 4, so the weight gradients differ by the order of FP32 sums alone: 2^-24 of the terms'
    # sizes per addition, sums of up to 4 * 68 * 40 terms of mixed sign that cancel by some 10^2
    import torch
    from paper_2607_16906_amd import hz
    net, _, gps, r = build(levels, base, W, H, 4)
    _, _, grad = hz.loss_backward(net, gps, r.reshape(-1), prec=prec)
    ref = torch.zeros_like(grad, dtype=torch.float64)
    for b in range(4):
        ref += hz.loss_backward(net, [gps[b]], r[b].contiguous(), prec=prec)[2].double() / 4
    for a, q in zip(per_layer(levels, base, grad), per_layer(levels, base, ref)):
        assert float((a - q).norm()) <= 1e-5 * float(q.norm())


@pytest.mark.gpu
@pytest.mark.parametrize("prec,tol", [("bf16", 0.1), ("fp32", 1e-3)])
@pytest.mark.parametrize("W,H", GRIDS)
@pytest.mark.parametrize("base", [16, 32, 64, 96])   # every channel tile of the kernels
def test_one_level_against_float64(base, W, H, prec, tol):
    # two 3x3 layers and the head. The error is that of the ReLU kinks: BF16 activations are off by some
    # 3e-3 of their spread, so 2e-3 of them change sides and with them sqrt(2e-3) = 5e-2 of the
    # gradient's norm per layer, two layers 7e-2 (FP32: 2^-24, sqrt(1e-7) = 3e-4). A wrong column at
    # the edge of a 16-pixel tile is sqrt(1 / 16) of its taps.
    from paper_2607_16906_amd import hz
    from oracle import helmholtz as ohz, unet
    from synth import C_REF
    import torch
    net, theta, gps, r = build(1, base, W, H, 2)
    _, _, grad = hz.loss_backward(net, gps, r.reshape(-1), prec=prec)
    if prec == "bf16":
        theta = torch.from_numpy(theta).to(torch.bfloat16).float().numpy()
    specs = unet.layer_specs(1, base, 5)
    ops = [ohz.Problem(np.float32(rng_for(89, 2, b).uniform(1400.0, 2800.0, H * W)).astype(np.float64).reshape(H, W), 2,
                       H_10PPW, 1.0, 2.0, C_REF) for b in range(2)]
    rr = r.cpu().numpy().astype(np.complex128).reshape(2, H, W)
    ref = torch.from_numpy(unet.loss_and_grad(theta.astype(np.float64), specs, ops, rr)[2]).cuda()
    for a, q in zip(per_layer(1, base, grad), per_layer(1, base, ref)):
        assert float((a - q).norm()) <= tol * float(q.norm())
