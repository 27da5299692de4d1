"""The coefficient kernel that shares a tile's bump values among samples
against the one that forms the sum per element (which the oracle tests cover at
a few samples): the same bits, over tiles that one, several and too many bumps
reach, partial tiles, sample counts that do not fill the last group, and random
variables that are not finite (they count only inside their disc)."""
import numpy as np
import pytest
import torch

from paper_1607_00693_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nfine,g,rho,N", [(16, 1, 0.7, 16400), (40, 3, 0.2, 1900), (64, 4, 0.25, 1030),
                                           (24, 2, 0.4, 20011), (50, 8, 0.125, 2055), (33, 5, 0.9, 2000),
                                           (256, 8, 0.125, 97)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_table_equals_direct(nfine, g, rho, N, dtype):
    from paper_1607_00693_amd import stomsfem as sm

    print(f"[coef] nfine={nfine} g={g} rho={rho} N={N} {dtype}", flush=True)
    prm = dict(g=g, rho=rho, eps=4.0 / nfine, base=2.0, amp=1.8, beta=0.5)
    xi = W.uniform_xi(N, g * g, 60 + nfine)
    xi[3, 0], xi[5, g * g - 1] = np.inf, np.nan
    xi = torch.from_numpy(xi).cuda()
    full = sm.coef_bumps(xi, nfine, **prm, dtype=dtype)
    tiles = ((nfine + 15) // 16) ** 2
    assert N * tiles // 8192 >= 2  # several samples per workgroup
    picks = [0, 1, 2, 3, 4, 5, 6, 31, 32, 33, N // 2, N - 2, N - 1]
    for s in picks:
        one = sm.coef_bumps(xi[s:s + 1].contiguous(), nfine, **prm, dtype=dtype)[0]
        assert torch.equal(torch.nan_to_num(full[s], nan=-7.0), torch.nan_to_num(one, nan=-7.0)), s
        assert torch.equal(torch.isnan(full[s]), torch.isnan(one)), s
