"""The launch choices a caller sees: autotuning reaches the last 3x3 layer of every width, and a variant
pinned for a level-0 layer is the launch that runs."""
import ctypes

import numpy as np
import pytest

from synth import H_10PPW, he_uniform, rng_for


def build(levels, base, nx, ny, npml=4):
    from paper_2607_16906_amd import hz
    net = hz.Net(levels, base, 5, he_uniform(hz.init_shapes(levels, base, 5), rng_for(103, 1, base)))
    n = (nx + 2 * npml) * (ny + 2 * npml)
    return net, hz.Problem(rng_for(103, 2, n).uniform(1400.0, 2800.0, n), nx, ny, npml, H_10PPW)


@pytest.mark.gpu
@pytest.mark.parametrize("base,prec", [(16, "bf16"), (32, "bf16"), (64, "bf16"), (96, "bf16"), (32, "fp32"),
                                       (40, "fp32"), (48, "fp32"), (96, "fp32"), (40, "fp64"), (48, "fp64")])
def test_last_layer_is_tuned(base, prec):
    # (40 channels are stored as 48; BF16 takes whole chunks of 32 channels or fewer, so not these two)
    from paper_2607_16906_amd import hz
    net, gp = build(2, base, 40, 24)
    net.autotune(gp, prec)
    last = len(hz.init_shapes(2, base, 5)) - 2
    _, _, cout, _ = net.layer_info(last)
    tn = net.layer_variant(last, 32, 48, prec=prec)[0]
    assert tn > 0 and cout % tn == 0


def workspace_after(net, gp, v):
    """The bytes an application leaves in a workspace of 0xff bytes, and its result."""
    import torch
    from paper_2607_16906_amd import hz
    lib = hz.load_library()
    z = torch.empty_like(v)
    ws = torch.full((lib.no_workspace_size(net.handle, gp.handle, hz.PREC["bf16"]),), 255, dtype=torch.uint8,
                    device="cuda")
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    assert lib.no_precond_apply(net.handle, gp.handle, hz.PREC["bf16"], hz.HZ_C64, p(v), p(z), p(ws),
                                ctypes.c_size_t(ws.numel()),
                                ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    torch.cuda.synchronize()
    return ws, z


@pytest.mark.gpu
@pytest.mark.parametrize("pins", [[0], [1], [0, 1]])
def test_pinned_encoder_layer_runs(pins):
    # level 0 in two launches keeps the first layer's output out of the workspace; a pinned layer runs by itself
    # and stores it
    check_pins(pins, enc=True)


@pytest.mark.gpu
@pytest.mark.parametrize("pins", [[-2], [-1], [-2, -1]])   # the decoder's two 3x3 layers
def test_pinned_decoder_layer_runs(pins):
    check_pins(pins, enc=False)


def check_pins(pins, enc):
    import torch
    from paper_2607_16906_amd import hz
    net, gp = build(3, 32, 40, 24)
    g = rng_for(103, 3, 0)
    v = torch.from_numpy(g.standard_normal(gp.n) + 1j * g.standard_normal(gp.n)).to(torch.complex64).cuda()
    last = len(hz.init_shapes(3, 32, 5)) - 2
    net.set_fused_upsampling(0)
    ws0, z0 = workspace_after(net, gp, v)
    net.set_fused_upsampling(2)
    ws2, z2 = workspace_after(net, gp, v)
    untouched = [int((w == 255).sum()) for w in (ws0, ws2)]
    assert untouched[1] > untouched[0] and torch.equal(z0, z2)   # the default mode stores less
    for k in pins:
        net.set_layer_variant(k if k >= 0 else last + 1 + k, 32, 48, 16, 8)
    ws, z = workspace_after(net, gp, v)
    assert torch.equal(z, z0)
    part = int((ws == 255).sum())
    assert part < untouched[1]
    if enc:   # the upsampled tensor is still missing (the decoder stores it and shares the encoder's temporary)
        assert part > untouched[0]
    for k in range(2) if not enc else (last - 1, last):   # the other half too: every tensor is stored
        net.set_layer_variant(k, 32, 48, 16, 8)
    ws, z = workspace_after(net, gp, v)
    assert torch.equal(z, z0) and torch.equal(ws, ws0)


@pytest.mark.gpu
def test_forms_with_the_head_give_the_staged_bits():
    # the last layer with the fused 1x1 head: the streamed forms that carry it (9 and 10 at 32 channels) against
    # the staged form, on grids around their 8- and 16-row tiles
    import torch
    from paper_2607_16906_amd import hz
    for nx, ny in ((40, 24), (5, 1), (9, 26), (70, 41)):
        net, gp = build(3, 32, nx, ny)
        net.set_fused_upsampling(0)
        Hp, Wp = (ny + 11) // 4 * 4, (nx + 11) // 4 * 4
        last = len(hz.init_shapes(3, 32, 5)) - 2
        g = rng_for(103, 4, nx)
        for prec in ("bf16", "fp32"):
            for dt in (torch.complex64, torch.complex128):
                v = torch.from_numpy(g.standard_normal(gp.n) + 1j * g.standard_normal(gp.n)).to(dt).cuda()
                net.set_layer_variant(last, Hp, Wp, 32, 8, prec=prec)
                ref = net.apply(gp, v, prec=prec)
                assert float(ref.abs().max()) > 0
                for fid, rows in ((9, 8), (10, 16)):
                    net.set_layer_variant(last, Hp, Wp, 32, rows, -fid, 1, prec=prec)
                    assert torch.equal(net.apply(gp, v, prec=prec), ref), (nx, ny, prec, fid)
