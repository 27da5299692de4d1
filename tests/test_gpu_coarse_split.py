"""Coarse systems with 33 to 64 elements per row, which are eliminated from both
ends: every remainder of the split (8 rows to a panel, B + 2 to B + 9 rows in the
middle), the smallest meshes that are split and those that are not, and a
pivot that is not positive in either end and in the middle.  U within 1e-10 of
the oracle's, as for the other coarse solves."""
import numpy as np
import pytest
import torch

from paper_1607_00693_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ncx,ncy", [(33, 2), (33, 3), (33, 4), (34, 3), (35, 5), (36, 4), (37, 3), (40, 9), (47, 4), (48, 7), (49, 3), (57, 6),
                                     (63, 3), (63, 5), (64, 2), (64, 3), (64, 4), (64, 70)])
def test_split_matches_oracle(orc, ncx, ncy):
    from paper_1607_00693_amd import stomsfem as sm

    print(f"[gpu-split] {ncx} x {ncy}", flush=True)
    N, m = 3, 2
    S, _, _ = orc.upscale(W.lognormal_field((N, ncy * m, ncx * m), 1.0, 2000 + ncx * 10 + ncy), ncx, ncy, m)
    Sd = torch.from_numpy(S).cuda()
    for load in (None, W.uniform_array((ncx * ncy, 4), 0.0, 1.0, 78)):
        U = sm.coarse_solve(Sd, ncx, ncy, load=None if load is None else torch.from_numpy(load).cuda())[0].cpu().numpy()
        ref, _, _ = orc.coarse_solve(S, ncx, ncy, load_vec=load)
        assert (np.abs(U - ref).max(1) <= 1e-10 * np.abs(ref).max(1)).all()


@pytest.mark.parametrize("row", [0, 10, 19, 38])
def test_bad_pivot_is_reported(row):
    from paper_1607_00693_amd import stomsfem as sm

    nc = 40
    q1 = torch.tensor([4, -1, -2, -1, 4, -1, -2, 4, -1, 4], dtype=torch.float64, device="cuda") / 6
    S = q1.repeat(3, nc * nc, 1)
    S[1, row * nc:(row + 2) * nc] *= -1.0
    st = torch.full((3,), 7, dtype=torch.int32, device="cuda")
    U = sm.coarse_solve(S.contiguous(), nc, nc, status=st)[0]
    assert st.tolist() == [sm.OK, sm.ENOTSPD, sm.OK]
    assert torch.isfinite(U[0]).all() and (U[0] - U[2]).abs().max() == 0
