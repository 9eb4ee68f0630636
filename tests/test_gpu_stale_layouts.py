"""The stale Boss / Assistant pipeline over the row layouts (one launch for both passes of a tick on the
64-lane ones up to 1024 floats, one each elsewhere) against the oracle's schedule."""
import numpy as np
import pytest
import torch

from paper_1905_03381_amd import api

import test_gpu_stale as stale
from gpu_util import clear_draws, dense_features, dev, host, scalar_dev

pytestmark = pytest.mark.gpu


# widths inside, at and past the edges of the shared launch; pools of one block, of several, and one
# that leaves a last pool of a single row; fewer steps than batches in the queue
@pytest.mark.parametrize("n,d,P,k", [(900, 132, 200, 1), (2401, 256, 600, 3), (1500, 508, 700, 2), (3001, 1000, 1000, 1),
                                     (700, 1024, 300, 5), (900, 1028, 400, 1), (600, 2052, 250, 2)])
def test_batches_and_model(ref, n, d, P, k):
    r = stale.rng(d)
    X = r.standard_normal((n, d)).astype(np.float32)
    X /= np.linalg.norm(X, axis=1, keepdims=True)
    y = np.where(X @ r.standard_normal(d) > 0, 1.0, -1.0).astype(np.float32)
    perm = r.permutation(n).astype(np.int32)
    w0, phi0 = np.zeros(d, np.float32), (0.5 * r.standard_normal(d)).astype(np.float32)
    gamma, lam, lr0, T, lr_a, step0 = 0.05, 1e-4, 1.0, 0.9, 2.0, 0
    for seed in range(11, 31):
        want = ref.train_stale(ref.Features.dense(X), y, perm, P, w0, phi0, 0.2, gamma, seed, step0, lam, lr0, T, lr_a, k)
        if all(clear_draws(ref, p, gamma, seed, step0 + s).all() for s, p in enumerate(want["prob"])):
            break
    F = dense_features(X)
    got = stale._run_gpu(F, y, perm, n, P, d, k, gamma, seed, step0, lam, lr0, T, lr_a, w0, phi0, 0.2, True)
    stale._compare(ref, got, want, P, gamma, seed, step0)
    # without a history the batches live in the workspace's ring: the same model, bit for bit
    ws, w, phi, b = api.Workspace(P, d, staleness=k), dev(w0), dev(phi0), scalar_dev(0.2)
    cfg = api.step_config(gamma, lam, lr0, lr_a, 0.0, seed, step0, scalar_dev(T))
    tu = torch.zeros(1, dtype=torch.int32, device="cuda")
    api.train_epoch_stale(F, dev(y), dev(perm), n, P, k, w, phi, b, cfg, tu, None, None, ws, torch.cuda.Stream())
    assert np.array_equal(host(w), got[0]) and np.array_equal(host(phi), got[1]) and float(host(b)[0]) == got[2]


def test_pools_beyond_direct_counting(ref):
    """Above 2^18 candidates a drawn pool is compacted by launches of its own behind the update."""
    n, d, P, k = 1000, 132, (1 << 18) + 5, 1
    r = stale.rng(d)
    X = r.standard_normal((n, d)).astype(np.float32)
    X /= np.linalg.norm(X, axis=1, keepdims=True)
    y = np.where(X @ r.standard_normal(d) > 0, 1.0, -1.0).astype(np.float32)
    perm = r.integers(0, n, 2 * P + 9).astype(np.int32)  # (rows come up again and again)
    w0, phi0 = np.zeros(d, np.float32), (0.5 * r.standard_normal(d)).astype(np.float32)
    gamma, lam, lr0, T, lr_a, step0 = 0.05, 1e-4, 1.0, 0.9, 2.0, 0
    for seed in range(11, 41):
        want = ref.train_stale(ref.Features.dense(X), y, perm, P, w0, phi0, 0.2, gamma, seed, step0, lam, lr0, T, lr_a, k)
        if all(clear_draws(ref, p, gamma, seed, step0 + s).all() for s, p in enumerate(want["prob"])):
            break
    got = stale._run_gpu(dense_features(X), y, perm, perm.size, P, d, k, gamma, seed, step0, lam, lr0, T, lr_a, w0, phi0, 0.2, True)
    stale._compare(ref, got, want, P, gamma, seed, step0)
