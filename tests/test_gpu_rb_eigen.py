"""The offline reduced basis at the edges of its eigen-solver: one unknown, 64
and 66 columns (where a lane takes more of a column), 126 and 129 (where the
matrix leaves LDS), primal and dual forms, the cell sizes where a lane of the
snapshot kernel takes more of a pivot (11, 16, 22), and training sets of few distinct
samples (a Gram matrix of rank 3).

Tolerances: r exact and the first eigenvalues within 1e-8 (1e-12 of the
largest), as for the 8 x 8 build; Z^T E Z = I within 1e-10 (columns of the
solver are orthogonal to 1e-14, E is conditioned below 1e4); and the KL
property Z^T E Psi Psi^T E Z = diag(lambda) within 1e-10 of the largest
eigenvalue (snapshots on both sides within 1e-13), which does not depend on
the gaps of the spectrum.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize(
    "m,ntrain,distinct",
    [(2, 1, 1), (2, 3, 3), (3, 1, 1), (3, 2, 2), (5, 40, 40), (6, 20, 20), (9, 22, 22), (9, 64, 2), (10, 40, 40), (12, 21, 21),
     (12, 22, 22), (12, 42, 42), (13, 42, 42), (13, 43, 43), (13, 50, 50), (13, 46, 2), (20, 16, 16), (11, 8, 8), (15, 5, 5), (16, 5, 5), (21, 4, 4), (22, 4, 4),
     (26, 3, 3)])
def test_modes_match_oracle(m, ntrain, distinct):
    from oracle import core, rb
    from paper_1607_00693_amd import stomsfem as sm

    print(f"[gpu-rb-eigen] m={m} ntrain={ntrain} distinct={distinct}", flush=True)
    ncx, ncy, nI = 2, 1, (m - 1) ** 2
    rng = np.random.default_rng(100 * m + ntrain)
    base = np.exp(0.5 * rng.standard_normal((distinct, ncy * m, ncx * m)))
    a = np.concatenate([base] * (ntrain // distinct + 1))[:ntrain].copy()
    model = sm.reduce(torch.from_numpy(a).cuda(), ncx, ncy, m, r_max=8, tail_tol=1e-6)
    r, lam, Z = model.export("r"), model.export("lambda"), model.export("Z")
    for K in range(ncx * ncy):
        blk = a[:, :, K * m:(K + 1) * m]
        om = rb.rb_offline(blk, r_max=8, tail_tol=1e-6)
        ref = np.zeros(nI)
        ref[:min(nI, len(om["sigma"]))] = om["sigma"][:nI] ** 2
        if distinct == 1:  # the centred snapshots are rounding: nothing but finite numbers to compare
            assert np.isfinite(lam[K]).all() and np.isfinite(Z[K]).all()
            continue
        assert r[K] == om["r"]
        np.testing.assert_allclose(lam[K, :8], ref[:8], rtol=1e-8, atol=1e-12 * ref[0])
        assert (np.diff(lam[K]) <= 0).all()
        phis = np.stack([core.cell_phi(blk[s], core.BC_LINEAR) for s in range(ntrain)])[:, :3, 1:-1, 1:-1].reshape(ntrain, 3, nI)
        Psi = (phis - phis.mean(axis=0)).transpose(2, 1, 0).reshape(nI, 3 * ntrain)
        E, _ = core.cell_system_dense(blk.mean(axis=0), core.BC_LINEAR)
        z = Z[K][:, :r[K]]
        assert not Z[K][:, r[K]:].any()
        assert np.abs(z.T @ E @ z - np.eye(r[K])).max() < 1e-10
        P = Psi.T @ (E @ z)
        assert np.abs(P.T @ P - np.diag(lam[K, :r[K]])).max() < 1e-10 * lam[K, 0]
    model.free()
