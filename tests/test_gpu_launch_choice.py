"""The launch choices a caller sees: autotuning reaches the last 3x3 layer of every width."""
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
