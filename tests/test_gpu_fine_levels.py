"""Fine solves by PCG over the shapes its kernels distinguish: a single level
(odd counts, below and above the 32 elements of the in-LDS levels), coarsest
levels in LDS and beyond, strip widths of 56, 60 and 62 columns and their
remainders, samples that converge at different iterations, one iteration only.

Tolerance: 1e-9 relative at a residual tolerance of 1e-13, as for the other
solves of this path.
"""
import numpy as np
import pytest
import torch

from oracle import twolevel

pytestmark = pytest.mark.gpu


def _coef(n, N, seed):
    a = np.exp(0.7 * np.random.default_rng(seed).standard_normal((N, n, n)))
    a[0] = 1.0  # converges in fewer iterations than the others
    return a


@pytest.mark.parametrize("n,N", [(2, 1), (3, 2), (5, 3), (7, 1), (8, 3), (9, 2), (12, 2), (16, 5), (31, 2), (32, 1), (33, 2), (34, 2), (48, 3),
                                 (56, 2), (57, 2), (60, 2), (64, 1), (66, 2), (113, 1), (120, 3), (122, 2), (124, 1), (126, 2), (168, 2)])
def test_levels_match_oracle(n, N):
    from paper_1607_00693_amd import stomsfem as sm

    print(f"[gpu-fine] n={n} N={N}", flush=True)
    a = _coef(n, N, 100 + n)
    u, it, st = sm.fine_solve_pcg(torch.from_numpy(a).cuda(), tol=1e-13)
    torch.cuda.synchronize()
    assert (st.cpu().numpy() == 0).all() and (it.cpu().numpy() >= 1).all()
    ref = twolevel.fine_solutions(a)
    got = u.cpu().numpy()
    for s in range(N):
        assert np.abs(got[s] - ref[s]).max() <= 1e-9 * np.abs(ref[s]).max(), s


def test_converged_samples_stay_and_one_iteration_is_reported():
    from paper_1607_00693_amd import stomsfem as sm

    a = _coef(128, 4, 7)
    a[2] *= np.exp(np.random.default_rng(8).uniform(-4, 4, (128, 128)))
    both, it, _ = sm.fine_solve_pcg(torch.from_numpy(a).cuda())
    it = it.cpu().numpy()
    assert it[0] < it[2]
    for s in range(4):  # a sample alone takes the same iterations; its sums group alike, so the bits differ by rounding only
        one, i1, _ = sm.fine_solve_pcg(torch.from_numpy(a[s:s + 1]).cuda())
        assert abs(int(i1[0]) - int(it[s])) <= 1
        assert (one[0] - both[s]).abs().max() <= 1e-9 * both[s].abs().max()
    _, i1, st = sm.fine_solve_pcg(torch.from_numpy(a).cuda(), max_iter=1)
    assert (i1.cpu().numpy() == 1).all() and (st.cpu().numpy() == sm.ENOCONV).all()
