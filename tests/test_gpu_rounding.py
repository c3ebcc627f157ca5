"""Device arithmetic that the kernels take for granted: the BF16 conversion is round-to-nearest-even for every
class of FP32 values, and the FP32 matrix instruction adds its products one after the other."""
import ctypes
import ctypes.util

import numpy as np
import pytest

from synth import he_uniform, rng_for


def bf16_rne(u):
    """FP32 bits to BF16 bits, round to nearest even (no NaN in u)."""
    u = u.astype(np.uint64)
    return ((u + 0x7fff + ((u >> 16) & 1)) >> 16).astype(np.uint16)


@pytest.mark.gpu
def test_bf16_stores_round_to_nearest_even():
    # a transposed layer of a zero input stores its FP32 biases: every upper half (all signs, exponents, subnormals
    # and infinities) with lower halves at, beside and far from the tie
    import torch
    from paper_2607_16906_amd import hz
    base = 256
    shapes = hz.init_shapes(2, base, 5)
    theta = torch.zeros(sum(int(np.prod(s)) + nb for s, _, nb in shapes), device="cuda")
    off = sum(int(np.prod(s)) + nb for s, _, nb in shapes[:4]) + int(np.prod(shapes[4][0]))
    net = hz.Net(2, base, 5, theta)
    kind, cin, cout, _ = net.layer_info(4)
    assert kind == 1 and cout == base
    x = torch.zeros((1, 1, 1, cin), device="cuda", dtype=torch.bfloat16)
    hi = np.arange(1 << 16, dtype=np.uint32) << 16
    for lo in (0, 1, 0x7fff, 0x8000, 0x8001, 0xffff):
        bits = hi | np.uint32(lo)
        vals = torch.from_numpy(bits.view(np.float32)).cuda()
        out = torch.empty((bits.size // base, 4, base), device="cuda", dtype=torch.bfloat16)
        for k in range(bits.size // base):
            theta[off:off + base] = vals[k * base:(k + 1) * base]
            net.set_weights(theta)
            net.layer_forward(4, x, out[k], H=1, W=1)
        got = out.view(torch.int16).cpu().numpy().view(np.uint16)
        assert (got == got[:, :1]).all()   # the four pixels of a channel
        got = got[:, 0].ravel()
        nan = ((bits & 0x7f800000) == 0x7f800000) & ((bits & 0x7fffff) != 0)
        zero = (bits & 0x7fffffff) == 0    # 0 + -0 is +0
        want = np.where(zero, 0, bf16_rne(np.where(nan, 0, bits)))
        assert np.array_equal(got[~nan], want[~nan])
        assert (((got[nan] & 0x7f80) == 0x7f80) & ((got[nan] & 0x7f) != 0)).all()   # NaN stays NaN


@pytest.mark.gpu
def test_bf16_weights_round_to_nearest_even():
    # the packed weights, read back one input channel at a time: normal values and ties (weight times one, the
    # other products zero)
    import torch
    from paper_2607_16906_amd import hz
    base = 64
    shapes = hz.init_shapes(2, base, 5)
    off = sum(int(np.prod(s)) + nb for s, _, nb in shapes[:4])
    n = int(np.prod(shapes[4][0]))
    g = rng_for(109, 1, 0)
    bits = g.integers(0, 1 << 32, n, dtype=np.uint64).astype(np.uint32)
    bits = (bits & 0x807fffff) | (g.integers(32, 224, n).astype(np.uint32) << 23)   # 2^-95 to 2^96
    bits[::3] = (bits[::3] & 0xffff0000) | 0x8000   # ties
    theta = np.zeros(sum(int(np.prod(s)) + nb for s, _, nb in shapes), np.float32)
    theta[off:off + n] = bits.view(np.float32)
    net = hz.Net(2, base, 5, theta)
    _, cin, cout, _ = net.layer_info(4)
    x = torch.eye(cin, device="cuda", dtype=torch.bfloat16).reshape(1, 1, cin, cin).contiguous()
    y = torch.empty((1, 2, 2 * cin, cout), device="cuda", dtype=torch.bfloat16)
    net.layer_forward(4, x, y, H=1, W=cin)
    got = y.view(torch.int16).cpu().numpy().view(np.uint16).reshape(2, cin, 2, cout).transpose(1, 3, 0, 2)
    assert np.array_equal(got.ravel(), bf16_rne(bits))


@pytest.mark.gpu
@pytest.mark.parametrize("scale", [1.0, 1e-15, 1e-21, 1e15])   # products of normal and of subnormal size
def test_fp32_products_are_added_in_order(scale):
    # a transposed layer in FP32 is a chain of fused multiply-adds over the input channels, then the bias
    import torch
    from paper_2607_16906_amd import hz
    fmaf = ctypes.CDLL(ctypes.util.find_library("m")).fmaf
    fmaf.restype, fmaf.argtypes = ctypes.c_float, [ctypes.c_float] * 3
    shapes = hz.init_shapes(2, 32, 5)
    theta = he_uniform(shapes, rng_for(109, 2, 0))
    off = sum(int(np.prod(s)) + nb for s, _, nb in shapes[:4])
    cin, cout = shapes[4][0][:2]
    g = rng_for(109, 3, 0)
    w = (g.standard_normal((cin, cout, 4)) * scale).astype(np.float32)
    theta[off:off + w.size] = w.ravel()
    theta[off + w.size:off + w.size + cout] = 0.0
    net = hz.Net(2, 32, 5, theta)
    xs = (g.standard_normal((8, cin)) * scale).astype(np.float32)
    x = torch.from_numpy(xs.reshape(1, 1, 8, cin)).cuda()
    y = torch.empty((1, 2, 16, cout), device="cuda")
    net.layer_forward(4, x, y, H=1, W=8, prec="fp32")
    got = y.cpu().numpy().reshape(2, 8, 2, cout)
    ref = np.zeros_like(got)
    for i in range(8):
        for co in range(cout):
            for ab in range(4):
                a = 0.0
                for c in range(cin):
                    a = fmaf(float(w[c, co, ab]), float(xs[i, c]), a)
                ref[ab >> 1, i, ab & 1, co] = a
    assert np.array_equal(got, ref)
