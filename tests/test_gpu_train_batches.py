"""Training steps where the minibatch wraps round the training set, against the
oracle's FP64 trajectory: sets smaller than, of and just above one minibatch,
with and without an order, the moments and the step count carried over a
second call.

Tolerance as for the five steps on one fixed minibatch: components whose
gradient stays above 1e-2 of the patch maximum at every step, within 2e-2 of
the learning rate (the FP32 gradient, within 1e-4 of the maximum, moves a
normalised update by at most 1e-2 of the rate per step); the loss of the last
minibatch within 1e-4 of its value (parameters within 2e-2 * 1e-3 of the
oracle's in the components that carry the gradient).
"""
import numpy as np
import pytest
import torch

from paper_1607_00693_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ntrain,ordered", [(1, False), (7, True), (31, True), (32, False), (33, False), (33, True), (100, True)])
def test_wrapped_minibatches_match_oracle(ntrain, ordered):
    from oracle import mlp
    from paper_1607_00693_amd import stomsfem as sm

    print(f"[gpu-train] ntrain={ntrain} ordered={ordered}", flush=True)
    wl = W.MESH8
    fam = sm.bump_family(wl)
    lv, nl = sm.local_vars_bumps(wl.nc, wl.nc, wl.m, fam)
    init = W.mlp_init(wl.M, 31)
    model = sm.mlp_create(wl.nc, wl.nc, wl.m, lv, init, fam, 1.0)
    xi = W.uniform_xi(ntrain, wl.nxi, 2304)
    S = W.uniform_array((ntrain, wl.M, 10), -2, 2, 2305)
    sm.mlp_set_data(model, torch.from_numpy(xi).cuda(), torch.from_numpy(S).cuda())
    mu, sd = sm.mlp_standardization(model)
    perm = W.permutation(ntrain, 2306) if ordered else None
    perm_d = torch.from_numpy(perm).cuda() if ordered else None
    loss = torch.zeros(wl.M, dtype=torch.float32, device="cuda")
    lr, calls = 1e-3, (2, 3)
    for k in calls:
        sm.mlp_train(model, k, lr, perm_d, loss)
    got = sm.mlp_params(model).cpu().numpy().astype(np.float64)
    loss = loss.cpu().numpy()
    for K in range(0, wl.M, 9):
        X = np.zeros((ntrain, 4))
        X[:, :nl[K]] = xi[:, lv[K, :nl[K]]]
        X = X.astype(np.float32).astype(np.float64)
        T = ((S[:, K] - mu[K]) / sd[K]).astype(np.float32).astype(np.float64)
        p = init[K].astype(np.float64)
        m1, m2, well = np.zeros_like(p), np.zeros_like(p), np.ones(p.shape, bool)
        for t in range(1, sum(calls) + 1):
            rows = (np.arange(32) + 32 * (t - 1)) % ntrain
            rows = perm[rows] if ordered else rows
            value, g = mlp.grad(p, X[rows], T[rows], 4)
            well &= np.abs(g) >= 1e-2 * np.abs(g).max()
            p, m1, m2 = mlp.adam_step(p, g, m1, m2, t, lr)
        d = np.abs(got[K] - p)
        assert well.sum() >= 100  # of 9940: the oracle's own count (with one sample the output biases lead the gradient)
        assert d[well].max() <= 2e-2 * lr, (K, d[well].max())
        assert abs(loss[K] - value) <= 1e-4 * value, (K, loss[K], value)
    model.free()
