"""Mean and variance of the coarse solutions around the sample counts where
their summation changes (16 wavefronts, one or two passes at 1024), against
torch's FP64 sums of the same U: sums of n values in another order, n u relative
to the largest term with n <= 2100, u = 1.1e-16."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nc,N", [(2, 1), (4, 1), (4, 15), (8, 16), (8, 17), (8, 64), (8, 65), (9, 1023), (9, 1024), (9, 1025), (9, 2100), (40, 3)])
def test_mean_and_variance(nc, N):
    from paper_1607_00693_amd import stomsfem as sm

    print(f"[gpu-qoi] nc={nc} N={N}", flush=True)
    q1 = torch.tensor([4, -1, -2, -1, 4, -1, -2, 4, -1, 4], dtype=torch.float64, device="cuda") / 6
    scale = torch.rand((N, nc * nc, 1), dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(N)) + 0.5
    U, mean, var = sm.coarse_solve((q1 * scale).contiguous(), nc, nc)[:3]
    tol = 2100 * 1.2e-16
    assert (mean - U.mean(0)).abs().max() <= tol * U.abs().max()
    assert (var - ((U * U).mean(0) - U.mean(0) ** 2)).abs().max() <= 4 * tol * (U * U).max()
