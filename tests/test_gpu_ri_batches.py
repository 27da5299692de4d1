"""A pair's interpolated stiffness does not depend on the number of samples in
the call: the same bits whether one or four wavefronts share the pair's table,
for tables of three variables and of four."""
import pytest
import torch

from paper_1607_00693_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nn", [3, 4, 5, 6, 7, 8, 9])
def test_interpolated_pairs_are_the_same_bits_in_any_batch(nn):
    from paper_1607_00693_amd import stomsfem as sm

    wl = W.MESH8
    fam = sm.bump_family(wl)
    lv, nl = sm.local_vars_bumps(wl.nc, wl.nc, wl.m, fam)
    model = sm.interp_build(wl.nc, wl.nc, wl.m, lv, fam, nn)
    xg = torch.from_numpy(W.uniform_xi(2112, wl.nxi, seed=1706)).cuda()
    print(f"[gpu-ri-batches] nn={nn}", flush=True)
    S, _ = sm.interp_apply(model, xg)
    for first, count in ((0, 1), (5, 63), (100, 64), (700, 65), (0, 1000)):
        S1, _ = sm.interp_apply(model, xg[first:first + count].contiguous())
        torch.cuda.synchronize()
        assert torch.equal(S1, S[first:first + count]), (first, count)
    assert max(nl) == 4
    model.free()


@pytest.mark.parametrize("oversample,terms", [(0, 4), (0, 3), (4, 3)])
def test_kl_pairs_are_the_same_bits_in_any_batch(oversample, terms):
    from paper_1607_00693_amd import stomsfem as sm

    nc, m, nn = 8, 8, 5
    mu, modes, _ = sm.local_kl(m + 2 * oversample, 1.0 / (nc * m), 1.0, 0.5 / nc, terms)
    model = sm.kl_interp_build(nc, nc, m, torch.from_numpy(mu).cuda(), torch.from_numpy(modes).cuda(), nn,
                               oversample=oversample)
    N = 1100
    xi = torch.from_numpy(W.uniform_array((N, nc * nc, terms), -2.9, 2.9, 1707)).cuda()
    kappa = torch.ones((N, nc * m, nc * m), dtype=torch.float64, device="cuda")
    print(f"[gpu-ri-batches] oversample={oversample} terms={terms}", flush=True)
    S, _ = sm.kl_interp_apply(model, xi, kappa)
    for n in (1, 65, 1000):
        S1, _ = sm.kl_interp_apply(model, xi[:n].contiguous(), kappa[:n].contiguous())
        torch.cuda.synchronize()
        assert torch.equal(S1, S[:n]), n
    model.free()
