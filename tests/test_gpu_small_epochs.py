"""GPU parity of epochs over small pools (one block runs all steps): every step against the oracle's step
from the GPU's previous state, then the epoch in one call, bit for bit."""
import numpy as np
import pytest
import torch

from paper_1905_03381_amd import api

from gpu_util import dense_features, dev, host, scalar_dev
from stepwise import check_epoch

pytestmark = pytest.mark.gpu


def _problem(n, d, ld=None):
    r = np.random.default_rng(d)
    X = r.standard_normal((n, ld or d)).astype(np.float32)
    X /= np.linalg.norm(X[:, :d], axis=1, keepdims=True)
    y = np.where(X[:, :d] @ r.standard_normal(d) > 0, 1.0, -1.0).astype(np.float32)
    return X, y, r.permutation(n).astype(np.int32), (0.8 * r.standard_normal(d)).astype(np.float32)


# every lane layout at its first and last width, pools on both sides of the numbers of turns a wave
# takes (16 waves of 4, 2 or 1 rows; 2, 4 or 8 turns) and of the largest pool (one row more takes
# the kernels of a launch per step), pools that leave waves without rows, last pools of one row
@pytest.mark.parametrize("d,P,n,ld", [(4, 17, 60, None), (64, 128, 300, None), (64, 129, 259, 68), (60, 512, 1025, None),
                                      (64, 513, 1100, None), (68, 64, 130, None), (128, 65, 196, None), (128, 256, 513, 132),
                                      (132, 1, 3, None), (132, 33, 100, None), (256, 128, 300, None), (256, 129, 300, None)])
@pytest.mark.parametrize("hard", [False, True])
def test_small_pools(ref, d, P, n, ld, hard):
    X, y, perm, w0 = _problem(n, d, ld)
    ws = api.Workspace(P, d)
    counts, _ = check_epoch(ref, ref.Features.dense(X, d=d), dense_features(X, d=d), y, perm, n, P, w0,
                            None if hard else w0[::-1].copy(), 0.1, gamma=0.0 if hard else 0.2, seed=5, step0=3, lam=1e-3,
                            lr0=0.5, lr_a=0.3, T=0.4, ws=ws, hard=hard)
    assert len(counts) == -(-n // P)


def test_epoch_of_more_steps_than_a_launch():
    """1050 pools of two rows in one call against the same pools in two calls; no history, no bias and a
    constant step size beside all of them."""
    d, P, n = 64, 2, 2100
    X, y, perm, w0 = _problem(n, d)
    F, yd, pd, ws, T = dense_features(X), dev(y), dev(perm), api.Workspace(P, d), scalar_dev(0.4)
    got = []
    for cuts in ([0, n], [0, 1998, n]):
        w, phi, b, tu = dev(w0), dev(w0), scalar_dev(0.1), scalar_dev(0, torch.int32)
        hist, ids = torch.zeros(n // P, dtype=torch.int32, device="cuda"), torch.zeros(n, dtype=torch.int32, device="cuda")
        plain = dev(w0), dev(w0)
        for lo, hi in zip(cuts, cuts[1:]):
            cfg = api.step_config(0.2, 1e-3, 0.5, 0.3, 0.01, 5, lo // P, T)
            api.train_epoch(F, yd, pd[lo:], hi - lo, P, w, phi, b, cfg, tu, hist[lo // P:], ws, ids[lo:])
            api.train_epoch(F, yd, pd[lo:], hi - lo, P, plain[0], plain[1], None, cfg, None, None, ws)
        got.append([host(v) for v in (w, phi, b, tu, hist, ids) + plain])
    assert all(np.array_equal(u, v) for u, v in zip(*got))
    hist, ids, tu = got[0][4], got[0][5], got[0][3]
    assert tu[0] == np.count_nonzero(hist) and 0 < tu[0] < n // P
    pools = perm.reshape(-1, P)
    for t in np.flatnonzero(hist == 1)[:50]:
        assert ids[t * P] in pools[t]
    assert np.array_equal(ids.reshape(-1, P)[hist == 2], pools[hist == 2])
    assert np.isfinite(got[0][6]).all() and not np.array_equal(got[0][6], w0)


def _epoch_and_steps(X, y, perm, P, w0, phi0, gamma, T):
    """(w, phi, kept counts) of one train_epoch call and of one fused_step call per pool."""
    n, d = X.shape
    F, yd, pd, ws, Td = dense_features(X), dev(y), dev(perm), api.Workspace(P, d), scalar_dev(T)
    steps = -(-n // P)
    hist = torch.zeros(steps, dtype=torch.int32, device="cuda")
    w, phi, b = dev(w0), dev(phi0), scalar_dev(0.0)
    api.train_epoch(F, yd, pd, n, P, w, phi, b, api.step_config(gamma, 1e-3, 0.5, 0.1, 0.0, 5, 0, Td), None, hist, ws)
    ws_, phis, bs, counts, cnt = dev(w0), dev(phi0), scalar_dev(0.0), [], scalar_dev(0, torch.int32)
    for t in range(steps):
        cfg = api.step_config(gamma, 1e-3, 0.5, 0.1, 0.0, 5, t, Td)
        api.fused_step(F, yd, pd[t * P:], min(P, n - t * P), ws_, phis, bs, cfg, None, None, None, None, None, None, cnt, ws)
        counts.append(int(host(cnt)[0]))
    return (host(w), host(phi), host(hist).tolist()), (host(ws_), host(phis), counts)


@pytest.mark.parametrize("d,P", [(132, 128), (200, 100), (256, 33)])
def test_rejected_rows_reach_no_sum_whatever_they_hold(d, P):
    """Rows with an infinite or NaN feature that are not kept: the model stays finite, as in single steps."""
    n = 3 * P
    X, y, perm, w0 = _problem(n, d)
    phi0 = w0[::-1].copy()
    phi0[0] = -1.0                       # an infinite x[0] scores -inf: never kept at gamma = 0
    X[:, 0] = 0.0                        # (and so no kept row moves phi[0])
    for t in range(3):
        X[perm[t * P + 1], 0] = np.inf
        X[perm[t * P + P // 2], 0] = np.nan
        X[perm[t * P + P - 1], 0] = np.inf
    epoch, steps = _epoch_and_steps(X, y, perm, P, w0, phi0, 0.0, 0.4)
    assert epoch[2] == steps[2] and min(epoch[2]) > 0
    for u, v in zip(epoch[:2], steps[:2]):
        assert np.isfinite(u).all()
        # (three steps, sums of at most 128 terms in two orders: 2e-6 per step is above their rounding)
        assert np.allclose(u, v, rtol=1e-5, atol=6e-6)


@pytest.mark.parametrize("d,P", [(132, 17), (200, 1), (256, 17)])
def test_infinite_feature_in_a_kept_row_counts_once(d, P):
    """A turn past the end of a wave's share re-reads its last row and adds nothing: an infinite
    feature there moves its column to an infinity, not to a NaN."""
    X, y, perm, w0 = _problem(P, d)
    phi0 = w0[::-1].copy()
    w0[0], phi0[0] = 1.0, -1.0
    X[:, 0] = 0.0
    X[perm[P - 1], 0], y[perm[P - 1]] = np.inf, -1.0  # margin -inf, score -inf: both coefficients are -1
    epoch, steps = _epoch_and_steps(X, y, perm, P, w0, phi0, 1.0, 0.4)
    assert epoch[2] == steps[2] == [P]
    assert epoch[0][0] == steps[0][0] == -np.inf and epoch[1][0] == steps[1][0] == np.inf
    assert np.isfinite(epoch[0][1:]).all() and np.isfinite(epoch[1][1:]).all()
