"""When a solve captures its restart cycle as a graph: for a cycle that may repeat, not for one that cannot."""
import numpy as np
import pytest

from synth import H_10PPW, rng_for


def system(nx, seed):
    import torch
    from paper_2607_16906_amd import hz
    n = (nx + 8) * (nx + 8)
    gp = hz.Problem(rng_for(107, 1, seed).uniform(1400.0, 2800.0, n), nx, nx, 4, H_10PPW)
    g = rng_for(107, 2, seed)
    return gp, torch.from_numpy(g.standard_normal(n) + 1j * g.standard_normal(n)).cuda()


@pytest.mark.gpu
def test_a_cycle_that_cannot_repeat_is_not_captured():
    # a solve of one cycle has no use for a graph of it; one called with the same arguments again and again gets
    # it in the third call, and every call has the same result
    import torch
    from paper_2607_16906_amd import hz
    gp, b = system(40, 0)
    out = torch.empty_like(b)
    ws = torch.empty(hz.fgmres_workspace_bytes(gp, None, 12, 12, "c128", "fp32"), dtype=torch.uint8, device="cuda")
    build, xs = [], []
    for _ in range(5):
        x, info = hz.fgmres(gp, b, m=12, tol=1e-14, maxit=12, krylov="c128", workspace=ws, out=out)
        assert info.its == 12
        build.append(info.phase_ms["build"])
        xs.append(x.clone())
    assert build[0] == 0 and build[1] == 0 and build[2] > 0 and build[3] == 0 and build[4] == 0, build
    assert all(torch.equal(x, xs[0]) for x in xs)


@pytest.mark.gpu
def test_cycles_that_may_repeat_are_captured_at_once():
    # two full cycles and a short last one, with the graph of the full one captured beside the first
    import torch
    from paper_2607_16906_amd import hz
    gp, b = system(41, 1)
    ws = torch.empty(hz.fgmres_workspace_bytes(gp, None, 10, 25, "c64", "fp32"), dtype=torch.uint8, device="cuda")
    x, info = hz.fgmres(gp, b, m=10, tol=1e-14, maxit=25, krylov="c64", workspace=ws)
    assert info.its == 25 and info.phase_ms["build"] > 0
    y, again = hz.fgmres(gp, b, m=10, tol=1e-14, maxit=25, krylov="c64", workspace=ws)
    assert torch.equal(x, y) and np.array_equal(info.hist, again.hist)


@pytest.mark.gpu
def test_batch_of_one_cycle_counts_no_capture():
    from paper_2607_16906_amd import hz
    sys_ = [system(nx, nx) for nx in (20, 33)]
    _, infos = hz.fgmres_batched([gp for gp, _ in sys_], [b for _, b in sys_], m=8, tol=1e-14, maxit=8, krylov="c64")
    assert all(i.its == 8 and i.phase_ms["build"] == 0 for i in infos)
