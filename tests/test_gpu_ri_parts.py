"""Random interpolation of small batches, where four wavefronts share a patch's
table: every pair as in a batch that is large enough for one wavefront each.
Both sum the same at most nn^4 products in another order: within nn^4 units
roundings of sums of the basis' absolute values (below 10), 1e-12 relative to max|S|;
pairs outside the box and the statuses exactly."""
import pytest
import torch

from paper_1607_00693_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nn", [4, 5, 6, 7])
def test_small_batches_equal_large_ones(nn):
    from paper_1607_00693_amd import stomsfem as sm

    wl = W.MESH8
    fam = sm.bump_family(wl)
    lv, nl = sm.local_vars_bumps(wl.nc, wl.nc, wl.m, fam)
    model = sm.interp_build(wl.nc, wl.nc, wl.m, lv, fam, nn)
    xi = W.uniform_xi(2112, wl.nxi, seed=1705)
    xi[3, :2] = 1.25
    xi[62] = -1.5
    xg = torch.from_numpy(xi).cuda()
    st = torch.full((2112, wl.M), -7, dtype=torch.int32, device="cuda")
    S, _ = sm.interp_apply(model, xg, status=st)
    outside = (st != 0).sum(1).cpu()
    for n in (1, 63, 64, 65, 1000):
        print(f"[gpu-ri-parts] nn={nn} n={n}", flush=True)
        s1 = torch.full((n, wl.M), -7, dtype=torch.int32, device="cuda")
        S1, nfb = sm.interp_apply(model, xg[:n].contiguous(), status=s1)
        torch.cuda.synchronize()
        assert torch.equal(s1, st[:n]) and nfb == int(outside[:n].sum())
        d = (S1 - S[:n]).abs().amax(-1) / S[:n].abs().amax(-1)
        assert float(d.max()) <= 1e-12
    assert int(outside.sum()) > 0 and sorted(set(nl.tolist()))[-1] >= 3
    model.free()
