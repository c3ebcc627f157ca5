"""Training gradients layer by layer against float64 on ragged grids, with a network whose ReLUs are all active:
what is left is rounding. Two levels of 32 channels have the layers 8 -> 32, 32 -> 32, 32 -> 64, 64 -> 64, the transposed
64 -> 32 and the concatenated 64 -> 32. And the data gradient's larger tiles against its smaller ones."""
import numpy as np
import pytest

from synth import H_10PPW, he_uniform, rng_for

# padded sizes: 8 and 16 columns and one group more, heights below, at and across the tiles
GRIDS = [(8, 8), (16, 12), (20, 36), (24, 16), (36, 20), (68, 40)]


def active_theta(levels, base):
    """Weights of a tenth of their usual spread on activations around 1; the head's so small that its output, whose
    rounding the operator would enlarge, does not matter beside the residual."""
    from paper_2607_16906_amd import hz
    shapes = hz.init_shapes(levels, base, 5)
    theta, off = he_uniform(shapes, rng_for(113, 1, base)), 0
    for k, (s, _, nb) in enumerate(shapes):
        n, head = int(np.prod(s)), k + 1 == len(shapes)
        theta[off:off + n] *= 1e-3 if head else 0.08
        theta[off + n:off + n + nb] = 0.0 if head else 1.0
        off += n + nb
    return theta, shapes


def fields(W, H, B):
    g = rng_for(113, 3, W)
    # a residual with a mean: the sums over the pixels do not cancel
    r = 1 + 0.5j + 0.3 * (g.standard_normal((B, H, W)) + 1j * g.standard_normal((B, H, W)))
    c = [np.float32(rng_for(113, 2, b).uniform(1400.0, 2800.0, (H, W))) for b in range(B)]
    return c, r.astype(np.complex64)


@pytest.mark.gpu
@pytest.mark.parametrize("prec,tol", [("bf16", 1e-2), ("fp32", 2e-5)])
@pytest.mark.parametrize("W,H", GRIDS)
@pytest.mark.parametrize("levels,base", [(2, 32), (2, 64), (3, 16)])
def test_layers_against_float64(levels, base, W, H, prec, tol):
    # BF16: activations and their gradients are rounded once per layer, by 2^-9 at most; of values this much alike
    # the roundings do not average out: 5 of them. FP32: sums of up to 2 * 68 * 40 terms of one sign, 2^-24 sqrt(5440)
    # = 4e-6, and what the layers pass on. One column too few of 68 is 1.5e-2.
    import torch
    from oracle import helmholtz as ohz, unet
    from paper_2607_16906_amd import hz
    from synth import C_REF
    theta, shapes = active_theta(levels, base)
    c, r = fields(W, H, 2)
    net = hz.Net(levels, base, 5, theta)
    gps = [hz.Problem(f.ravel(), W - 4, H - 4, 2, H_10PPW) for f in c]
    _, _, grad = hz.loss_backward(net, gps, torch.from_numpy(r.reshape(2, -1)).cuda(), prec=prec)
    if prec == "bf16":
        theta = torch.from_numpy(theta).to(torch.bfloat16).float().numpy()
    ops = [ohz.Problem(f.astype(np.float64), 2, H_10PPW, 1.0, 2.0, C_REF) for f in c]
    ref = unet.loss_and_grad(theta.astype(np.float64), unet.layer_specs(levels, base, 5), ops,
                             r.astype(np.complex128))[2]
    got, off = grad.double().cpu().numpy(), 0
    for k, (s, _, nb) in enumerate(shapes):
        for n in (int(np.prod(s)), nb):
            e = np.linalg.norm(got[off:off + n] - ref[off:off + n]) / np.linalg.norm(ref[off:off + n])
            assert e <= tol, (k, n, e)
            off += n


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["bf16", "fp32"])
def test_large_batch_is_the_mean_of_its_samples(prec):
    # 64 samples of 64 x 60 take the data gradient's large tiles (rows of 8 and 16, 32 and 64 channels, split and
    # not), one sample the smallest: the same activation gradients up to the exact factor 1 / 64, so the weight
    # gradients differ by the order of FP32 sums of terms of one sign alone
    import torch
    from paper_2607_16906_amd import hz
    B, W, H = 64, 64, 60
    theta, shapes = active_theta(3, 32)
    c, r = fields(W, H, B)
    net = hz.Net(3, 32, 5, theta)
    gps = [hz.Problem(f.ravel(), W - 4, H - 4, 2, H_10PPW) for f in c]
    rd = torch.from_numpy(r.reshape(B, -1)).cuda()
    _, per, grad = hz.loss_backward(net, gps, rd, prec=prec)
    ref = torch.zeros_like(grad, dtype=torch.float64)
    one = torch.empty_like(per)
    for b in range(B):
        _, p, g = hz.loss_backward(net, [gps[b]], rd[b].contiguous(), prec=prec)
        ref += g.double() / B
        one[b] = p[0]
    assert torch.equal(one, per)
    off = 0
    for s, _, nb in shapes:
        for n in (int(np.prod(s)), nb):
            a, q = grad[off:off + n].double(), ref[off:off + n]
            assert float((a - q).norm()) <= 1e-5 * float(q.norm()), n
            off += n
