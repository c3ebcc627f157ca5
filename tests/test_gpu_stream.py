"""Streamed-weights 3x3 layers (net_stream.h) through the C ABI: every form gives the staged form's bits."""
import numpy as np
import pytest

from synth import he_uniform, rng_for

# id: (16-channel blocks per wavefront, rows per wavefront, wavefronts along channels / rows)
FORMS = {1: (1, 2, 4, 1), 2: (1, 4, 4, 1), 3: (1, 8, 4, 1), 4: (2, 8, 4, 1), 5: (1, 4, 2, 2), 6: (1, 8, 2, 2),
         7: (2, 4, 2, 2), 8: (2, 8, 2, 2), 9: (2, 2, 1, 4), 10: (2, 4, 1, 4), 11: (1, 2, 2, 2), 12: (1, 2, 1, 4),
         13: (1, 4, 1, 4)}
# layer of a 3-level, 32-channel network: 1 (32 -> 32, pooled), 5 (128 -> 128, no concatenation),
# 7 (128 -> 64, two input parts)
LAYERS = [1, 5, 7]
# a single pixel row / column, one less and one more than the 16-wide tile and the 2- to 16-row tiles
SIZES = [(1, 1, 2), (2, 18, 1), (14, 16, 2), (18, 34, 1)]


def _net():
    from paper_2607_16906_amd import hz
    theta = he_uniform(hz.init_shapes(3, 32, 5), rng_for(77, 2, 0))
    return hz.Net(3, 32, 5, theta)


def _tensors(net, layer, H, W, B, dtype):
    import torch
    _, cin, cout, cat = net.layer_info(layer)
    rng = rng_for(77, 3, 1000 * layer + 10 * H + W)
    mk = lambda c: torch.from_numpy(np.maximum(rng.standard_normal((B, H, W, c)), -0.5)).to("cuda").to(dtype)
    x0 = mk(cat if cat else cin)
    x1 = mk(cin - cat) if cat else None
    y = torch.empty((B, H, W, cout), device="cuda", dtype=dtype)
    pool = torch.empty((B, H // 2, W // 2, cout), device="cuda", dtype=dtype) if H % 2 == 0 and W % 2 == 0 else None
    return x0, x1, y, pool


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["bf16", "fp32"])
@pytest.mark.parametrize("H,W,B", SIZES)
@pytest.mark.parametrize("layer", LAYERS)
def test_forms_give_the_staged_bits(layer, H, W, B, prec):
    import torch
    from paper_2607_16906_amd import hz
    net = _net()
    x0, x1, y, pool = _tensors(net, layer, H, W, B, {"bf16": torch.bfloat16, "fp32": torch.float32}[prec])
    run = lambda: net.layer_forward(layer, x0, y, H=H, W=W, batch=B, x1=x1, pool=pool, prec=prec)
    net.set_layer_variant(layer, H, W, 16, 8, batch=B, prec=prec)
    run()
    ref = (y.clone(), pool.clone() if pool is not None else None)
    seen = 0
    for fid, (ncb, rpw, wc, wr) in FORMS.items():
        tn, rows = 16 * ncb * wc, rpw * wr
        if ref[0].shape[-1] % tn:
            with pytest.raises(hz.HzError):
                net.set_layer_variant(layer, H, W, tn, rows, -fid, 1, batch=B, prec=prec)
            continue
        net.set_layer_variant(layer, H, W, tn, rows, -fid, 1, batch=B, prec=prec)
        assert net.layer_variant(layer, H, W, batch=B, prec=prec) == (tn, rows, -fid, 1)
        y.fill_(float("nan"))
        run()
        assert torch.equal(y, ref[0]), fid
        if pool is not None:
            assert torch.equal(pool, ref[1]), fid
        seen += 1
    assert seen >= 7
