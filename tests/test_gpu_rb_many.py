"""The offline reduced basis of many small patches: at least 256 of them (the Gram
matrices in one part, several coefficients of the element table to a thread), and
patches of one and four unknowns, whose Gram matrices have a kernel of their own
(fewer and more snapshots than a wavefront has lanes, one sample, the dual form).

Tolerances as for the other builds: r exact, eigenvalues within 1e-8 (1e-12 of
the largest), and S of the online stage within 1e-10 of the oracle's, with which
the modes and the table enter.  And patches of one unknown take no longer than
1.3 times the same mesh in patches of nine (1.65 times before)."""
import numpy as np
import pytest
import torch

from paper_1607_00693_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ncx,ncy,m,ntrain", [(2, 1, 2, 9), (2, 1, 3, 2), (2, 1, 3, 30), (32, 16, 2, 5), (32, 16, 2, 70), (16, 17, 3, 8),
                                              (32, 16, 4, 9), (16, 16, 5, 24), (85, 3, 5, 24), (20, 13, 8, 40), (33, 40, 6, 3)])
def test_builds_match_oracle(ncx, ncy, m, ntrain):
    from oracle import rb
    from paper_1607_00693_amd import stomsfem as sm

    print(f"[gpu-rb-many] {ncx} x {ncy} m={m} ntrain={ntrain}", flush=True)
    a = W.lognormal_field((ntrain + 2, ncy * m, ncx * m), 0.5, 5000 + 10 * m + ntrain)
    model = sm.reduce(torch.from_numpy(a[:ntrain].copy()).cuda(), ncx, ncy, m, r_max=8, tail_tol=1e-6)
    S = sm.reduce_apply(model, torch.from_numpy(a[ntrain:].copy()).cuda(), precision=sm.PREC_F64).cpu().numpy()
    r, lam, nI = model.export("r"), model.export("lambda"), (m - 1) ** 2
    for K in sorted({0, 1, ncx * ncy // 2, ncx * ncy - 1}):
        blk = a[:, K // ncx * m:(K // ncx + 1) * m, K % ncx * m:(K % ncx + 1) * m]
        om = rb.rb_offline(blk[:ntrain], r_max=8, tail_tol=1e-6)
        ref = np.zeros(nI)
        ref[:min(nI, len(om["sigma"]))] = om["sigma"][:nI] ** 2
        assert r[K] == om["r"]
        np.testing.assert_allclose(lam[K, :8], ref[:8], rtol=1e-8, atol=1e-12 * ref[0])
        for s in range(2):
            want = rb.rb_online_S(om, blk[ntrain + s])
            assert np.abs(S[s, K] - want).max() <= 1e-10 * np.abs(want).max(), (K, s)
    model.free()


def test_patches_of_one_unknown_cost_little_more_than_of_nine():
    from paper_1607_00693_amd import stomsfem as sm

    a = torch.from_numpy(W.uniform_array((30, 256, 256), 0.5, 2.0, 5001)).cuda()

    def time(m):
        best = float("inf")
        for _ in range(7):
            t0, t1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            t0.record()
            sm.reduce(a, 256 // m, 256 // m, m).free()
            t1.record()
            torch.cuda.synchronize()
            best = min(best, t0.elapsed_time(t1))
        return best

    time(2), time(4)
    assert time(2) <= 1.3 * time(4)
