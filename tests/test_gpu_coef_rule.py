"""Which coefficient kernel a batch takes.  The kernel that shares a tile's bump
values among samples gives the bits of the one that forms the sum per element,
over batches large enough for it (partial last groups, tiles that one to sixteen
bumps reach, discs of one and of two cells, random variables that are not
finite), and a batch that is a little larger does not cost much more: 1100
samples of 64 x 64 took 2.4 times as long as 1000."""
import numpy as np
import pytest
import torch

from paper_1607_00693_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nfine,g,rho,N", [(16, 1, 0.7, 65549), (40, 3, 0.2, 8001), (64, 4, 0.25, 4500), (64, 4, 0.25, 20011),
                                           (24, 2, 0.4, 20011), (50, 8, 0.125, 9001), (256, 8, 0.125, 330),
                                           (48, 4, 0.5, 6007), (48, 4, 0.5, 30011), (512, 12, 0.1, 99)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_batch_equals_single_samples(nfine, g, rho, N, dtype):
    from paper_1607_00693_amd import stomsfem as sm

    print(f"[coef-rule] nfine={nfine} g={g} rho={rho} N={N} {dtype}", flush=True)
    prm = dict(g=g, rho=rho, eps=4.0 / nfine, base=2.0, amp=1.8, beta=0.5)
    xi = W.uniform_xi(N, g * g, 70 + nfine)
    xi[N // 3, 0], xi[N // 2, g * g - 1] = np.inf, np.nan
    xi = torch.from_numpy(xi).cuda()
    full = sm.coef_bumps(xi, nfine, **prm, dtype=dtype)
    for s in (0, 1, 31, 32, 33, N // 3, N // 3 + 1, N // 2, N - 2, N - 1):
        one = sm.coef_bumps(xi[s:s + 1].contiguous(), nfine, **prm, dtype=dtype)[0]
        assert torch.equal(torch.nan_to_num(full[s], nan=-7.0), torch.nan_to_num(one, nan=-7.0)), s
        assert torch.equal(torch.isnan(full[s]), torch.isnan(one)), s


@pytest.mark.parametrize("nfine,g,rho,few,more", [(64, 4, 0.25, 1000, 1100), (64, 8, 0.5, 1000, 1100), (1024, 8, 0.5, 3, 4)])
def test_a_larger_batch_costs_in_proportion(nfine, g, rho, few, more):
    from paper_1607_00693_amd import stomsfem as sm

    def time(N):
        xi = torch.from_numpy(W.uniform_xi(N, g * g, 71)).cuda()
        out = torch.empty((N, nfine, nfine), dtype=torch.float64, device="cuda")
        best = float("inf")
        for _ in range(7):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(20):
                sm.coef_bumps(xi, nfine, g, rho, 4.0 / nfine, out=out)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    assert time(more) <= 1.5 * more / few * time(few)
