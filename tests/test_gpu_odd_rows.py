"""GPU parity of dense rows that do not fill a register layout: rows that end inside one, and rows none
takes -- wider than 2048, or a width, leading dimension or address off 16 bytes -- at the edges of
their kernels' pieces."""
import numpy as np
import pytest
import torch

from paper_1905_03381_amd import api

import test_gpu_dense as dense
import test_gpu_sk as sk
from gpu_util import dense_features

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ws():
    return api.Workspace(4000, 9000)


# a block of 512 threads owns 2048 columns per piece: one column either side of each number of
# pieces, widths of every remainder by four, padded and odd leading dimensions, and pools that give
# some blocks no row, one row, and more than a register set of them
# -- and below that a row per wave, one layout up to 256, 512 and 1024 floats
SHAPES = [(20, 3, None, 20), (40, 4, 5, 33), (300, 5, None, 300), (300, 63, None, 260), (300, 255, None, 255),
          (300, 256, 257, 280), (600, 257, None, 590), (300, 511, None, 129), (300, 513, 514, 300), (600, 1023, None, 520),
          (40, 1025, None, 33), (300, 1027, 1029, 300), (300, 2047, None, 257), (64, 2049, None, 64),
          (300, 2050, 2052, 255), (600, 4095, None, 520), (40, 4096, 4096, 40), (600, 4097, 4099, 513),
          (300, 6144, None, 256), (1500, 6145, None, 1400), (300, 8191, None, 300), (20, 8192, None, 1),
          (20, 8193, None, 20), (3300, 1367, None, 3300)]


@pytest.mark.parametrize("n,d,ld,P", SHAPES)
def test_odd_rows_match_the_oracle(ref, ws, n, d, ld, P):
    dense.test_assistant_score(ref, n, d, ld, P, True)
    dense.test_fused_step_matches_oracle_step(ref, ws, n, d, ld, P, 0.1)
    dense.test_svm_sgd_step(ref, ws, n, d, ld, min(P, 300), False)
    dense.test_assistant_update(ref, ws, n, d, ld, P)
    r = dense.rng(7)
    X = r.standard_normal((n, ld or d)).astype(np.float32)
    X /= np.linalg.norm(X[:, :d], axis=1, keepdims=True)
    y = np.where(r.random(n) < 0.5, 1.0, -1.0).astype(np.float32)
    idx = r.permutation(n)[:P].astype(np.int32)
    sk._run_and_check(ref, ws, ref.Features.dense(X, d=d), dense_features(X, d=d), y, idx, P, d, 0.4)


# rows that end inside a 64-lane layout, and pools on both sides of the switches between the numbers
# of rows a wave requests at once
@pytest.mark.parametrize("d,P", [(132, 1), (132, 4097), (252, 16_385), (256, 4096), (256, 16_400), (260, 700), (508, 4097),
                                 (516, 513), (1020, 300), (1028, 400), (2044, 65)])
def test_whole_step_on_rows_inside_a_layout(ref, d, P):
    n, big = P + 3, api.Workspace(P + 3, d)
    dense.test_fused_step_matches_oracle_step(ref, big, n, d, None, P, 0.1)
    r = dense.rng(7)
    X = r.standard_normal((n, d)).astype(np.float32)
    X /= np.linalg.norm(X, axis=1, keepdims=True)
    y = np.where(r.random(n) < 0.5, 1.0, -1.0).astype(np.float32)
    idx = r.permutation(n)[:P].astype(np.int32)
    sk._run_and_check(ref, big, ref.Features.dense(X), dense_features(X), y, idx, P, d, 0.4)


@pytest.mark.parametrize("d,P", [(260, 300), (1020, 5000)])
def test_epoch_on_rows_inside_a_layout_is_its_steps(d, P):
    """One call per epoch (compaction carried by the next pass) against one call per step: same bits."""
    n = 3 * P + P // 3
    g = torch.Generator().manual_seed(d)
    X = torch.randn(n, d, generator=g)
    F = api.Features.dense((X / X.norm(dim=1, keepdim=True)).cuda())
    y = (2.0 * torch.randint(0, 2, (n,), generator=g) - 1.0).cuda()
    perm = torch.randperm(n, generator=g).to(torch.int32).cuda()
    T, work = torch.full((1,), 0.3, device="cuda"), api.Workspace(P, d)
    got = []
    for calls in ([(0, n)], [(lo, min(P, n - lo)) for lo in range(0, n, P)]):
        w, phi, b = torch.ones(d, device="cuda"), torch.ones(d, device="cuda"), torch.zeros(1, device="cuda")
        t = torch.zeros(1, dtype=torch.int32, device="cuda")
        hist = torch.zeros(4, dtype=torch.int32, device="cuda")
        ids, loss = torch.zeros(4 * P, dtype=torch.int32, device="cuda"), torch.zeros(4 * P, device="cuda")
        for lo, count in calls:
            cfg = api.step_config(0.1, 1e-3, 2.0, 0.3, 0.0, 5, lo // P, T)
            api.train_epoch(F, y, perm[lo:], count, P, w, phi, b, cfg, t, hist[lo // P:], work, ids[lo:], loss[lo:])
        got.append((w, phi, b, t, hist, ids, loss))
    assert all(torch.equal(u, v) for u, v in zip(*got))
    assert 0 < got[0][4].min() and got[0][4][0] < P


@pytest.mark.parametrize("d", [7, 130, 1023, 1027, 4097])
def test_odd_rows_with_infinities_in_the_last_columns(ws, d):
    """The last columns of a row that is no whole number of pieces are read twice and count once:
    an infinite value there gives an infinite score, not a NaN, and reaches no other row."""
    P = 9
    X = torch.randn(P, d, generator=torch.Generator().manual_seed(d)).cuda()
    X[3, d - 2] = float("inf")
    phi = torch.full((d,), 0.01, device="cuda")
    logit, prob = torch.zeros(P, device="cuda"), torch.zeros(P, device="cuda")
    api.assistant_score(api.Features.dense(X), None, P, phi, None, logit, prob)
    assert logit[3].item() == float("inf") and prob[3].item() == 1.0
    rest = torch.arange(P, device="cuda") != 3
    want = (X[rest].double().cpu() @ phi.double().cpu()).float().cuda()
    # (a sum of d terms of size 0.01: rounding below 1e-5)
    assert torch.all((logit[rest] - want).abs() <= 1e-5)


def _one_step(X, y, w0, phi0, hard, gamma, T):
    """w and phi (None with hard thresholds) after one whole step on all rows."""
    n, d = X.shape
    work, F, yd = api.Workspace(n, d), dense_features(X), dense.dev(y)
    w, phi, cnt = dense.dev(w0), dense.dev(phi0), dense.scalar_dev(0, torch.int32)
    if hard:
        api.sk_step(F, yd, None, n, w, dense.scalar_dev(T), 0.0, 1.0, None, None, None, None, None, cnt, work)
        return dense.host(w), None
    cfg = api.step_config(gamma, 0.0, 1.0, 1.0, 0.0, 3, 0, dense.scalar_dev(T))
    api.fused_step(F, yd, None, n, w, phi, None, cfg, None, None, None, None, None, None, cnt, work)
    return dense.host(w), dense.host(phi)


@pytest.mark.parametrize("d", [7, 130, 785, 1023, 1027, 4137, 9000])
@pytest.mark.parametrize("hard", [False, True])
@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_rows_without_a_gradient_add_nothing(d, hard, bad):
    """A row whose coefficients are zero (not kept, or kept with its margin met and its score right) adds
    nothing, whatever it holds: the same model as with a large finite value in the place of the bad one."""
    n, r = 21, dense.rng(d)
    X = (r.standard_normal((n, d)) / np.sqrt(d)).astype(np.float32)
    y = np.where(r.random(n) < 0.5, 1.0, -1.0).astype(np.float32)
    w0, phi0 = r.standard_normal(d).astype(np.float32), r.standard_normal(d).astype(np.float32)
    w0[0], phi0[0], X[:, 0] = 1.0, -1.0, 0.0
    got = []
    for value in (1e30, bad):  # margin beyond 1 and probability 0 (a NaN row is never kept: gamma < 1)
        for row in (4, n - 1):
            X[row, 0], y[row] = value, 1.0
        got.append(_one_step(X, y, w0, phi0, hard, 0.0 if np.isnan(bad) else 1.0, 0.4))
    assert np.isfinite(got[0][0]).all() and np.array_equal(got[0][0], got[1][0])
    if not hard:
        assert np.isfinite(got[0][1]).all() and np.array_equal(got[0][1], got[1][1])


@pytest.mark.parametrize("d", [130, 132, 256, 1020, 1024, 1027])
def test_infinite_feature_in_the_last_row_counts_once(d):
    """A place past the last row re-reads it and adds nothing: an infinite feature there moves its
    column to an infinity, not to a NaN."""
    X = np.zeros((1, d), np.float32)
    X[0, 0] = np.inf
    w = _one_step(X, np.full(1, -1.0, np.float32), np.ones(d, np.float32), None, True, 0.0, 0.4)[0]
    assert w[0] == -np.inf and np.array_equal(w[1:], np.ones(d - 1, np.float32))


@pytest.mark.parametrize("d", [4097, 4137, 6145, 8192])
@pytest.mark.parametrize("P", [1024, 3000])
def test_sums_past_4096_columns_are_rounded_once(d, P):
    """Passes that update both vectors keep the sums of the columns from 4096 on in doubles until all
    blocks are added up: a one beside terms of 2^24 that cancel between two blocks is not lost."""
    X, cols = np.zeros((P, d), np.float32), np.unique([4096, 4096 + (d - 4096) // 2, d - 1])
    for c in cols:
        X[0, c], X[1, c], X[P - 1, c] = 2.0 ** 24, 1.0, -2.0 ** 24
    zero = np.zeros(d, np.float32)
    # (w = phi = 0: every margin is 0 and every score 1/2; T = 2 makes every label 0)
    w, phi = _one_step(X, np.ones(P, np.float32), zero, zero, False, 1.0, 2.0)
    inv = np.float32(1.0) / np.float32(P)
    assert np.all(w[cols] == inv) and np.all(phi[cols] == -np.float32(0.5) * inv)
    assert np.count_nonzero(w) == np.count_nonzero(phi) == cols.size


@pytest.mark.parametrize("d", [1027, 2050, 4137, 8001])
def test_scores_out_of_matrices_of_any_size(d):
    """Scoring takes plain or non-temporal loads by the size of the whole matrix (76 and 256 MB are the
    limits): the same bits from all of them, and the sum of the products."""
    n, P = (1 << 26) // d + 300, 277
    X = torch.empty(n, d, device="cuda").normal_(generator=torch.Generator(device="cuda").manual_seed(d))
    phi = torch.randn(d, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1)) / d ** 0.5
    got = []
    for rows in (X, X[:n // 2], X[:300]):  # 257 to 266, 128 to 133 and 1 to 10 MB
        logit, prob = torch.zeros(P, device="cuda"), torch.zeros(P, device="cuda")
        api.assistant_score(api.Features.dense(rows), None, P, phi, None, logit, prob)
        got.append((logit, prob))
    assert all(torch.equal(got[0][k], other[k]) for other in got[1:] for k in (0, 1))
    want = X[:P].double().cpu() @ phi.double().cpu()
    scale = X[:P].double().cpu().abs() @ phi.double().cpu().abs()
    assert torch.all((got[0][0].cpu() - want).abs() <= 1e-5 * scale)


# rows of a block around the numbers of rows a batch of each layout works on at once (8, 4, 4 and 1 for
# one to four pieces a thread) and around a group of 64
@pytest.mark.parametrize("per_block", [4, 7, 8, 9, 16, 20, 31, 32, 40, 63, 64])
@pytest.mark.parametrize("d", [5, 130, 132, 1000, 1025, 2049, 4097, 6145, 9000])
def test_every_row_of_a_block_has_its_own_draw(ref, d, per_block):
    """Keep flags against the scores that the same call returns and the uniforms of the definition, in the
    scoring call and in the whole step."""
    n, P, gamma, seed, step = 300, 256 * per_block + 100, 0.05, 9, 4
    g = torch.Generator(device="cuda").manual_seed(d)
    F = api.Features.dense(torch.randn(n, d, device="cuda", generator=g) / d ** 0.5)
    idx = torch.randint(0, n, (P,), device="cuda", generator=g, dtype=torch.int32)
    y = torch.ones(n, device="cuda")
    w, phi, work = torch.zeros(d, device="cuda"), torch.randn(d, device="cuda", generator=g), api.Workspace(P, d)
    u = torch.from_numpy(ref.uniforms(seed, step, P)).cuda().double()
    for whole in (False, True):
        prob, keep = torch.zeros(P, device="cuda"), torch.full((P,), 9, dtype=torch.uint8, device="cuda")
        pos, cnt = torch.zeros(P, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
        if whole:
            cfg = api.step_config(gamma, 0.0, 0.1, 0.1, 0.0, seed, step, dense.scalar_dev(0.4))
            api.fused_step(F, y, idx, P, w, phi, None, cfg, None, prob, keep, pos, None, None, cnt, work)
        else:
            api.score_shrink(F, idx, P, phi, None, gamma, seed, step, None, prob, keep, pos, cnt, work)
        p = gamma + (1.0 - gamma) * prob.double()
        sure = (u - p).abs() > 1e-6
        assert torch.equal(keep[sure].bool(), (u < p)[sure]) and int(cnt) == int(keep.sum())
        assert torch.equal(pos[:int(cnt)].long(), torch.nonzero(keep).view(-1))


@pytest.mark.parametrize("d", [5, 7, 130, 785, 1023, 1027, 2050, 4097, 6147, 9001])
@pytest.mark.parametrize("back", [1, 2, 3, 4, 5])
def test_infinite_model_entries_in_the_last_columns(d, back):
    """An infinite entry of the model among the last columns of an odd row, which are read twice, gives
    infinite scores and losses with the signs of the features, as anywhere else."""
    P = 9
    X = torch.randn(P, d, generator=torch.Generator().manual_seed(d)).cuda()
    v = torch.full((d,), 0.01, device="cuda")
    v[d - back] = float("inf")
    F, sign = api.Features.dense(X), torch.sign(X[:, d - back])
    logit, prob = torch.zeros(P, device="cuda"), torch.zeros(P, device="cuda")
    api.assistant_score(F, None, P, v, None, logit, prob)
    assert torch.equal(logit, sign * float("inf"))
    loss, cnt = torch.zeros(P, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    api.sk_step(F, torch.ones(P, device="cuda"), None, P, v.clone(), dense.scalar_dev(0.5), 0.0, 0.0, loss, None, None, None,
                None, cnt, api.Workspace(P, d))
    assert torch.equal(loss, torch.where(sign > 0, 0.0, float("inf"))) and int(cnt) == int((sign < 0).sum())
