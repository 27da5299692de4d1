"""A sample's fine solution does not depend on the batch it is solved in: the
same bits and the same iterations alone, in a small batch and past the 64
samples of a chunk.  The sizes have one level and several, strips and
remainders of 8 rows, and segments whose length changes with the batch."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [33, 75, 100, 128, 196, 258])
def test_solutions_are_the_same_bits_in_any_batch(n):
    from paper_1607_00693_amd import stomsfem as sm

    N = 67
    a = np.exp(0.7 * np.random.default_rng(900 + n).standard_normal((N, n, n)))
    a[0] = 1.0  # converges in fewer iterations than the others
    ag = torch.from_numpy(a).cuda()
    print(f"[gpu-fine-batches] n={n}", flush=True)
    u, it, st = sm.fine_solve_pcg(ag)
    assert not st.any()
    for first, count in ((0, 1), (1, 1), (3, 4), (20, 17), (63, 4), (66, 1)):
        part = slice(first, first + count)
        u1, it1, _ = sm.fine_solve_pcg(ag[part].contiguous())
        torch.cuda.synchronize()
        assert torch.equal(it1, it[part]), (first, count)
        assert torch.equal(u1, u[part]), (first, count)
