"""Petrov-Galerkin coarse systems at the sizes where a lane takes more of a
pivot's square (8, 11, 16 and 21 elements per row and the next), with a single
unknown per row or column and more rows than the ring of element rows, against
the oracle: non-symmetric element matrices (a K_Q1 plus a perturbation with zero
row sums), U within 1e-10."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ncx,ncy", [(2, 9), (3, 2), (3, 12), (8, 9), (9, 8), (11, 5), (12, 12), (16, 3), (17, 17), (21, 20), (22, 7), (32, 9)])
def test_sizes_match_oracle(orc, ncx, ncy):
    from paper_1607_00693_amd import stomsfem as sm

    print(f"[gpu-pg] {ncx} x {ncy}", flush=True)
    N = 3
    rng = np.random.default_rng(1500 + 70 * ncx + ncy)
    A = rng.uniform(0.3, 4.0, size=(N, ncx * ncy, 1, 1))
    E = rng.normal(size=(N, ncx * ncy, 4, 4)) * 0.15 * A
    E -= E.mean(axis=3, keepdims=True)
    S16 = (A * orc.q1_kref() + E).reshape(N, ncx * ncy, 16)
    load = rng.uniform(0.5, 1.5, size=(ncx * ncy, 4))
    U = sm.coarse_solve_pg(torch.from_numpy(S16).cuda(), ncx, ncy, load=torch.from_numpy(load).cuda())[0].cpu().numpy()
    ref, _, _ = orc.coarse_solve_pg(S16, ncx, ncy, load.reshape(-1))
    assert (np.linalg.norm(U - ref, axis=1) <= 1e-10 * np.linalg.norm(ref, axis=1)).all()
