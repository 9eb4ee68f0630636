"""GPU parity of the CSR path (sparse linear-SVM and token-list shapes) against the oracle."""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

from paper_1905_03381_amd import api, synth

from gpu_util import (RTOL, abs_dot_scale, assert_close_scaled, assert_logit_prob, clear_draws,
                      csr_features, dev, host, kernel_constant, scalar_dev)

pytestmark = pytest.mark.gpu

# The kernel that scores with the head of phi in LDS: its columns, the rows it takes over more than TABLE_MIN_COLS columns (and
# at most twice TABLE_COLS), and over fewer.
TABLE_COLS = kernel_constant("kScoreTableCols")
TABLE_MIN_COLS = kernel_constant("kScoreTableMinCols")
TABLE_ROWS = kernel_constant("kScoreTableMinRows")
TABLE_MANY_ROWS = kernel_constant("kScoreTableManyRows")


def rng(seed):
    return np.random.default_rng(seed)


@pytest.fixture(scope="module")
def sparse():
    """Down-scaled sparse config: 30,000 rows, d = 2^16, about 100 entries per row."""
    rowptr, col, val, y, _ = synth.sparse_svm(n=30_000, d=1 << 16, mean_nnz=100, threads=4)
    return rowptr, col, val, y, 1 << 16


@pytest.fixture(scope="module")
def ws():
    return api.Workspace(1 << 16, 1 << 16)


def test_csr_score_and_fused_keep(ref, ws, sparse):
    rowptr, col, val, y, d = sparse
    n = rowptr.size - 1
    P = 20_000
    r = rng(1)
    phi = (3.0 * r.standard_normal(d)).astype(np.float32)
    idx = r.permutation(n)[:P].astype(np.int32)
    Fh = ref.Features.csr(rowptr, col, val, d)
    F = csr_features(rowptr, col, val, d)
    ref_logit, ref_prob = ref.assistant_score(Fh, idx, P, phi, bias=0.3)
    S = abs_dot_scale(Fh, idx, phi)
    logit, prob = torch.zeros(P, device="cuda"), torch.zeros(P, device="cuda")
    api.assistant_score(F, dev(idx), P, dev(phi), scalar_dev(0.3), logit, prob)
    assert_logit_prob(host(logit), host(prob), ref_logit, ref_prob, S, bias=0.3)
    gamma, seed, step = 0.1, 3, 8
    keep_ref, _ = ref.shrink(ref_prob, gamma, seed, step)
    keep = torch.zeros(P, dtype=torch.uint8, device="cuda")
    pos = torch.full((P,), -1, dtype=torch.int32, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int32, device="cuda")
    api.score_shrink(F, dev(idx), P, dev(phi), scalar_dev(0.3), gamma, seed, step, None, prob, keep,
                     pos, cnt, ws)
    k = host(keep)
    clear = clear_draws(ref, ref_prob, gamma, seed, step)
    assert np.array_equal(k[clear], keep_ref[clear])
    m = int(host(cnt)[0])
    assert m == int(k.sum()) and np.array_equal(host(pos)[:m], np.flatnonzero(k))


@pytest.mark.parametrize("ones", [False, True])
@pytest.mark.parametrize("indexed", [True, False])
def test_csr_score_large_pool_equals_small_pools(ref, ws, ones, indexed):
    """Large pools are scored by the kernel that keeps the head of phi in LDS, smaller ones by the general
    kernel: both add a row's terms in the same order, so one pool and the same rows in pools of a fifth give the same
    bits -- and the oracle's values.  Rows of 0 to 260 entries: half of them exceed the 128
    entries of the first kernel's main loop and take its walk over long rows; a fifth of the
    columns lie past its table."""
    P, d = TABLE_ROWS + 617, TABLE_COLS + TABLE_COLS // 4
    n, part = P + 5000, P // 5
    assert TABLE_MIN_COLS < d <= 2 * TABLE_COLS and part < TABLE_ROWS
    r = rng(41)
    lens = r.integers(0, 261, size=n)
    rowptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(lens, out=rowptr[1:])
    col = r.integers(0, d, size=int(rowptr[-1])).astype(np.int32)
    val = (r.standard_normal(col.size) / 10.0).astype(np.float32)
    phi = r.standard_normal(d).astype(np.float32)
    idx = r.permutation(n)[:P].astype(np.int32) if indexed else None
    Fh = ref.Features.csr(rowptr, col, None if ones else val, d)
    F = csr_features(rowptr, col, None if ones else val, d)
    lens = lens[idx if indexed else slice(0, P)]
    assert (lens > 128).mean() > 0.3 and (lens <= 128).mean() > 0.3 and (lens == 0).sum() > 10
    bias, gamma, seed, step = scalar_dev(-0.4), 0.2, 11, 6
    logit, prob = torch.zeros(P, device="cuda"), torch.zeros(P, device="cuda")
    api.assistant_score(F, None if idx is None else dev(idx), P, dev(phi), bias, logit, prob)
    ids = idx if indexed else np.arange(P, dtype=np.int32)
    ref_logit, ref_prob = ref.assistant_score(Fh, ids, P, phi, bias=-0.4)
    assert_logit_prob(host(logit), host(prob), ref_logit, ref_prob, abs_dot_scale(Fh, ids, phi), bias=-0.4)
    logit2, prob2 = torch.zeros(P, device="cuda"), torch.zeros(P, device="cuda")
    for lo in range(0, P, part):
        m = min(part, P - lo)
        api.assistant_score(F, dev(ids[lo:lo + m]), m, dev(phi), bias, logit2[lo:], prob2[lo:])
    assert np.array_equal(host(logit), host(logit2)) and np.array_equal(host(prob), host(prob2))
    # keep flags of the fused score + keep + compact call: same draws, same probabilities
    keep = torch.zeros(P, dtype=torch.uint8, device="cuda")
    pos = torch.full((P,), -1, dtype=torch.int32, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int32, device="cuda")
    prob3 = torch.zeros(P, device="cuda")
    api.score_shrink(F, None if idx is None else dev(idx), P, dev(phi), bias, gamma, seed, step, None,
                     prob3, keep, pos, cnt, ws)
    assert np.array_equal(host(prob3), host(prob))
    keep_ref, _ = ref.shrink(ref_prob, gamma, seed, step)
    clear = clear_draws(ref, ref_prob, gamma, seed, step)
    k = host(keep)
    assert np.array_equal(k[clear], keep_ref[clear])
    m = int(host(cnt)[0])
    assert m == int(k.sum()) and np.array_equal(host(pos)[:m], np.flatnonzero(k))


@pytest.mark.parametrize("ones", [True, False])
@pytest.mark.parametrize("P", [5_000, TABLE_MANY_ROWS + 37])
def test_csr_score_row_ends(ref, ones, P):
    """Rows are read four entries at a time, the last piece ending with the row: rows of every length
    around the pieces (0 to 9, 61 to 68, 125 to 133 entries), the shortest first, where nothing lies before
    them in the matrix -- through the general kernel (5000 rows) and through the one with phi in
    LDS, which takes over at more rows of so few columns.  No row holds column 0, whose model entry
    is infinite: what a piece shares with another row or entry must not count."""
    lens = np.tile(np.r_[1, 1, 0, 0:10, 61:69, 125:134, 5, 3, 2], P // 33 + 1)[:P]
    r, d = rng(43), 3000
    rowptr = np.zeros(P + 1, dtype=np.int64)
    np.cumsum(lens, out=rowptr[1:])
    col = r.integers(1, d, size=int(rowptr[-1])).astype(np.int32)
    val = None if ones else (r.standard_normal(col.size) / 10.0).astype(np.float32)
    phi = r.standard_normal(d).astype(np.float32)
    Fh = ref.Features.csr(rowptr, col, val, d)
    ref_logit, ref_prob = ref.assistant_score(Fh, None, P, phi, bias=0.2)
    scale = abs_dot_scale(Fh, np.arange(P), phi)
    phi[0] = np.inf
    logit, prob = torch.zeros(P, device="cuda"), torch.zeros(P, device="cuda")
    api.assistant_score(csr_features(rowptr, col, val, d), None, P, dev(phi), scalar_dev(0.2), logit, prob)
    assert_logit_prob(host(logit), host(prob), ref_logit, ref_prob, scale, bias=0.2)


def _device_time(call, n=10):
    """Shortest of five runs of n calls, in milliseconds."""
    call()
    best = float("inf")
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(n):
            call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


@pytest.mark.parametrize("ones", [True, False])
def test_csr_score_long_rows_in_a_large_pool(ref, ones):
    """Rows of more than 128 entries (up to 700) in a pool that the kernel with phi in LDS takes: the bits of the
    general kernel's scores of the halves, and about their time (four times that when such rows were walked
    one by one)."""
    P, d = TABLE_MANY_ROWS, 2000
    r = rng(47)
    lens = r.integers(129, 400, size=P)
    lens[::1000] = r.integers(400, 701, size=lens[::1000].size)
    rowptr = np.zeros(P + 1, dtype=np.int64)
    np.cumsum(lens, out=rowptr[1:])
    col = r.integers(0, d, size=int(rowptr[-1])).astype(np.int32)
    val = None if ones else (r.standard_normal(col.size) / 16.0).astype(np.float32)
    F, phi, bias = csr_features(rowptr, col, val, d), dev(r.standard_normal(d).astype(np.float32)), scalar_dev(0.2)
    out = [torch.zeros(P, device="cuda") for _ in range(4)]
    ids = torch.arange(P, dtype=torch.int32, device="cuda")
    half = P // 2

    def halves():
        for lo in (0, half):
            api.assistant_score(F, ids[lo:], half, phi, bias, out[2][lo:], out[3][lo:])
    whole = _device_time(lambda: api.assistant_score(F, ids, P, phi, bias, out[0], out[1]))
    split = _device_time(halves)
    assert np.array_equal(host(out[0]), host(out[2])) and np.array_equal(host(out[1]), host(out[3]))
    assert whole < 1.5 * split, (whole, split)


def test_csr_all_ones_values(ref, ws):
    """Token lists: val == NULL means every entry is 1; repeated tokens add."""
    rowptr, col, val, len_s, len_t, d = synth.sentence_pairs(n=5000, vocab=2000)
    r = rng(2)
    phi = (0.2 * r.standard_normal(d)).astype(np.float32)
    Fh = ref.Features.csr(rowptr, col, None, d)
    F = csr_features(rowptr, col, None, d)
    P = 5000
    ref_logit, ref_prob = ref.assistant_score(Fh, None, P, phi)
    logit, prob = torch.zeros(P, device="cuda"), torch.zeros(P, device="cuda")
    api.assistant_score(F, None, P, dev(phi), None, logit, prob)
    assert_logit_prob(host(logit), host(prob), ref_logit, ref_prob, abs_dot_scale(Fh, np.arange(P), phi))
    # with the length features as values
    Fh2 = ref.Features.csr(rowptr, col, val, d)
    F2 = csr_features(rowptr, col, val, d)
    ref_logit, ref_prob = ref.assistant_score(Fh2, None, P, phi, bias=-0.5)
    api.assistant_score(F2, None, P, dev(phi), scalar_dev(-0.5), logit, prob)
    assert_logit_prob(host(logit), host(prob), ref_logit, ref_prob,
                      abs_dot_scale(Fh2, np.arange(P), phi), bias=-0.5)


def _dots(Fh, ids, v):
    """x_r . v for the listed CSR rows, float64, by scipy."""
    S = sp.csr_matrix((Fh.val.astype(np.float64), Fh.col, Fh.rowptr), shape=(Fh.n, Fh.d))
    return S[np.asarray(ids)] @ v.astype(np.float64)


def _col_abs_sum(Fh, ids, d):
    out = np.zeros(d)
    for i in ids:
        lo, hi = Fh.rowptr[i], Fh.rowptr[i + 1]
        v = np.ones(hi - lo) if Fh.val is None else np.abs(Fh.val[lo:hi].astype(np.float64))
        np.add.at(out, Fh.col[lo:hi], v)
    return out


def test_csr_svm_step_and_assistant_update(ref, ws, sparse):
    rowptr, col, val, y, d = sparse
    n = rowptr.size - 1
    m = 3000
    r = rng(3)
    w0 = (2.0 * r.standard_normal(d)).astype(np.float32)
    phi0 = r.standard_normal(d).astype(np.float32)
    rows = r.permutation(n)[:m].astype(np.int32)
    Fh = ref.Features.csr(rowptr, col, val, d)
    F = csr_features(rowptr, col, val, d)
    lam, lr, T, lr_a, b0 = 1e-3, 0.5, 0.3, 0.2, 0.1
    w_ref, loss_ref = ref.svm_sgd_step(Fh, y, rows, m, w0, lam, lr)
    S = abs_dot_scale(Fh, rows, w0)
    dots = _dots(Fh, rows, w0) * y[rows]
    assert np.all(np.abs(dots - 1) > RTOL * S)
    w = dev(w0)
    loss = torch.zeros(m, device="cuda")
    api.svm_sgd_step(F, dev(y), dev(rows), scalar_dev(m, torch.int32), m, w, lam, lr, 0.0, loss, ws)
    assert_close_scaled(host(loss), loss_ref, S, "loss")
    absx = _col_abs_sum(Fh, rows[dots < 1], d)
    assert_close_scaled(host(w), w_ref, np.abs(w0.astype(np.float64)) + lr / m * absx, "w")
    phi_ref, b_ref = ref.assistant_update(Fh, rows, m, loss_ref, T, phi0, b0, lr_a)
    phi, b = dev(phi0), scalar_dev(b0)
    api.assistant_update(F, dev(rows), scalar_dev(m, torch.int32), m, dev(loss_ref), scalar_dev(T),
                         phi, b, lr_a, 0.0, ws)
    absx = _col_abs_sum(Fh, rows, d)
    assert_close_scaled(host(phi), phi_ref, np.abs(phi0.astype(np.float64)) + lr_a / m * absx, "phi")
    assert abs(float(host(b)[0]) - b_ref) <= RTOL * (abs(b0) + lr_a)
    # m = 0 leaves everything alone
    w = dev(w0)
    api.svm_sgd_step(F, dev(y), dev(rows), scalar_dev(0, torch.int32), m, w, lam, lr, 0.0, None, ws)
    assert np.array_equal(host(w), w0)


def test_csr_fused_step(ref, ws, sparse):
    rowptr, col, val, y, d = sparse
    n = rowptr.size - 1
    P = 8000
    r = rng(4)
    w0 = (2.0 * r.standard_normal(d)).astype(np.float32)
    phi0 = (2.0 * r.standard_normal(d)).astype(np.float32)
    idx = r.permutation(n)[:P].astype(np.int32)
    Fh = ref.Features.csr(rowptr, col, val, d)
    F = csr_features(rowptr, col, val, d)
    b0, gamma, step, lam, lr, T, lr_a = 0.0, 0.1, 3, 1e-3, 0.5, 0.1, 0.3
    for seed in range(1, 20):   # first Philox key with no draw inside the rounding band
        out = ref.step(Fh, y, idx, P, w0, phi0, b0, gamma, seed, step, lam, lr, T, lr_a)
        if clear_draws(ref, out["prob"], gamma, seed, step).all():
            break
    else:
        raise AssertionError("no clear seed")
    kept = out["kept_ids"]
    dots = _dots(Fh, kept, w0) * y[kept]
    # rows whose margin sits within rounding of the hinge kink may fall on either side
    on_kink = np.abs(dots - 1) <= RTOL * abs_dot_scale(Fh, kept, w0)
    assert on_kink.sum() <= 3
    w, phi, b = dev(w0), dev(phi0), scalar_dev(b0)
    Tt = scalar_dev(T)
    cfg = api.step_config(gamma, lam, lr, lr_a, 0.0, seed, step, Tt)
    prob = torch.zeros(P, device="cuda")
    keep = torch.zeros(P, dtype=torch.uint8, device="cuda")
    pos = torch.zeros(P, dtype=torch.int32, device="cuda")
    ids = torch.zeros(P, dtype=torch.int32, device="cuda")
    loss = torch.zeros(P, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int32, device="cuda")
    api.fused_step(F, dev(y), dev(idx), P, w, phi, b, cfg, None, prob, keep, pos, ids, loss, cnt, ws)
    m = out["m"]
    assert int(host(cnt)[0]) == m
    assert np.array_equal(host(keep), out["keep"])
    assert np.array_equal(host(pos)[:m], out["kept_pos"])
    assert np.array_equal(host(ids)[:m], out["kept_ids"])
    assert_close_scaled(host(loss)[:m], out["loss"], abs_dot_scale(Fh, kept, w0), "loss")
    absx_a = _col_abs_sum(Fh, kept[dots < 1], d)
    assert_close_scaled(host(w), out["w"], np.abs(w0.astype(np.float64)) + lr / m * absx_a, "w",
                        atol=lr / m * _col_abs_sum(Fh, kept[on_kink], d))
    absx = _col_abs_sum(Fh, kept, d)
    assert_close_scaled(host(phi), out["phi"], np.abs(phi0.astype(np.float64)) + lr_a / m * absx,
                        "phi")


@pytest.mark.parametrize("ones", [True, False])
@pytest.mark.parametrize("d", [3000, 20_000, 300_000])
def test_csr_fused_scores_have_the_bits_of_separate_ones(d, ones):
    """The whole-step pass and the scoring kernels add a row's terms in the same order (20,000 columns: the kernel
    with phi in LDS): same logits, probabilities and draws for rows on both sides of 64 and 128 entries,
    long ones, and short ones at the matrix's start, before fewer and more rows than a wave's lane groups."""
    n, many = 20_000, TABLE_ROWS + 13  # (rows of the matrix; places of the large pool, some rows there more than once)
    assert TABLE_MIN_COLS < 20_000
    r = rng(53)
    lens = np.where(r.random(n) < 0.5, r.integers(0, 70, size=n), r.integers(60, 300, size=n))
    lens[:4] = 1, 1, 0, 1
    rowptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(lens, out=rowptr[1:])
    col = r.integers(0, d, size=int(rowptr[-1])).astype(np.int32)
    val = None if ones else (r.standard_normal(col.size) / 8.0).astype(np.float32)
    F = csr_features(rowptr, col, val, d)
    y, idx = dev(np.where(r.random(n) < 0.5, -1.0, 1.0).astype(np.float32)), dev(np.resize(r.permutation(n), many).astype(np.int32))
    phi = dev((r.standard_normal(d) / (8.0 if ones else 1.0)).astype(np.float32))
    cfg = api.step_config(0.1, 1e-3, 0.5, 0.3, 0.0, 7, 2, scalar_dev(0.1))
    for P, ids in ((many, idx), (300, idx), (40, None)):
        ws = api.Workspace(P, d)
        got = [torch.zeros(P, device="cuda") for _ in range(5)]
        keep = [torch.zeros(P, dtype=torch.uint8, device="cuda") for _ in range(2)]
        pos, kept = (torch.zeros(P, dtype=torch.int32, device="cuda") for _ in range(2))
        cnt = torch.zeros(1, dtype=torch.int32, device="cuda")
        api.score_shrink(F, ids, P, phi, scalar_dev(-0.2), 0.1, 7, 2, got[0], got[1], keep[0], pos, cnt, ws)
        api.fused_step(F, y, ids, P, torch.zeros(d, device="cuda"), phi.clone(), scalar_dev(-0.2), cfg, got[2], got[3],
                       keep[1], pos, kept, got[4], cnt, ws)
        assert np.array_equal(host(got[0]), host(got[2])) and np.array_equal(host(got[1]), host(got[3]))
        assert np.array_equal(host(keep[0]), host(keep[1]))


def _bits(t):
    return host(t).view(np.uint32).copy()


def test_csr_fused_steps_repeat_bit_for_bit(ws, sparse):
    """Five chained whole steps on the sparse shape, run four times from the same state: model,
    bias and losses come out with the same bits every time.  (Entries of a column reach its
    total by three routes -- the block's table, a hashed slot, a record -- and which route an
    entry takes depends on timing; every route adds in doubles and rounds once.)"""
    rowptr, col, val, y, d = sparse
    n, P, steps = rowptr.size - 1, 6000, 5
    r = rng(31)
    w0 = r.standard_normal(d).astype(np.float32)
    phi0 = r.standard_normal(d).astype(np.float32)
    perm = dev(r.permutation(n)[:steps * P].astype(np.int32))
    F = csr_features(rowptr, col, val, d)
    yd, Tt = dev(y), scalar_dev(0.3)
    cfg = api.step_config(0.1, 1e-3, 0.5, 0.3, 0.0, 5, 0, Tt)

    def run():
        w, phi, b = dev(w0), dev(phi0), scalar_dev(0.1)
        hist = torch.zeros(steps, dtype=torch.int32, device="cuda")
        loss = torch.full((steps, P), -3.0, device="cuda")
        api.train_epoch(F, yd, perm, steps * P, P, w, phi, b, cfg, None, hist, ws, None, loss)
        return _bits(w), _bits(phi), _bits(b), _bits(loss), host(hist).tolist()

    first = run()
    assert min(first[4]) > 500 and not np.array_equal(first[0], w0.view(np.uint32))
    for _ in range(3):
        again = run()
        assert again[4] == first[4]
        for name, x0, x1 in zip(("w", "phi", "bias", "losses"), first, again):
            assert np.array_equal(x0, x1), f"{name} differs between two runs of the same steps"


def test_gather_csr(ref, ws, sparse):
    rowptr, col, val, y, d = sparse
    n = rowptr.size - 1
    P = 5000
    r = rng(5)
    idx = r.permutation(n)[:P].astype(np.int32)
    kept_pos = np.sort(r.choice(P, 2100, replace=False)).astype(np.int32)
    Fh = ref.Features.csr(rowptr, col, val, d)
    F = csr_features(rowptr, col, val, d)
    cap = int(np.diff(rowptr)[idx[kept_pos]].sum())
    want_ptr, want_col, want_val = ref.gather_csr(Fh, idx, kept_pos, cap)
    out_ptr = torch.full((P + 1,), -1, dtype=torch.int64, device="cuda")
    out_col = torch.full((cap,), -1, dtype=torch.int32, device="cuda")
    out_val = torch.full((cap,), -1.0, device="cuda")
    pos_d = torch.zeros(P, dtype=torch.int32, device="cuda")
    pos_d[:2100] = dev(kept_pos)
    api.gather_csr(F, dev(idx), pos_d, scalar_dev(2100, torch.int32), P, out_ptr, out_col, out_val,
                   cap, ws)
    assert np.array_equal(host(out_ptr)[:2101], want_ptr)
    assert np.array_equal(host(out_col), want_col) and np.array_equal(host(out_val), want_val)
    # capacity too small: row pointers complete, rows past the capacity not copied
    small = cap // 2
    out_col2 = torch.full((small,), -1, dtype=torch.int32, device="cuda")
    out_val2 = torch.full((small,), -1.0, device="cuda")
    api.gather_csr(F, dev(idx), pos_d, scalar_dev(2100, torch.int32), P, out_ptr, out_col2, out_val2,
                   small, ws)
    ptr = host(out_ptr)[:2101]
    assert np.array_equal(ptr, want_ptr) and ptr[-1] > small
    fits = int(np.searchsorted(want_ptr, small, side="right") - 1)
    assert np.array_equal(host(out_col2)[:want_ptr[fits]], want_col[:want_ptr[fits]])
    assert np.all(host(out_col2)[want_ptr[fits]:] == -1)
    # one entry short: only the last kept row stays out, nothing is written past the capacity
    # (the buffers hold one guard entry behind it)
    out_col3 = torch.full((cap,), -1, dtype=torch.int32, device="cuda")
    out_val3 = torch.full((cap,), -1.0, device="cuda")
    api.gather_csr(F, dev(idx), pos_d, scalar_dev(2100, torch.int32), P, out_ptr, out_col3, out_val3,
                   cap - 1, ws)
    assert np.array_equal(host(out_ptr)[:2101], want_ptr)
    last = want_ptr[2099]
    assert np.array_equal(host(out_col3)[:last], want_col[:last])
    assert np.array_equal(host(out_val3)[:last], want_val[:last])
    assert np.all(host(out_col3)[last:] == -1) and np.all(host(out_val3)[last:] == -1.0)


def test_sparse_config_full_size_first_pools(ref):
    """The sparse linear-SVM configuration at full size (n = 2,000,000, d = 2^20, about 100
    entries per row, pools of 65,536): two chained whole steps against the oracle."""
    n, d, P = 2_000_000, 1 << 20, 65536
    rowptr, col, val, y, _ = synth.sparse_svm(n=n, d=d, threads=16)
    Fh = ref.Features.csr(rowptr, col, val, d)
    F = csr_features(rowptr, col, val, d)
    ws = api.Workspace(P, d)
    perm = synth.epoch_permutation(n, seed=7, epoch=0)
    gamma, seed, lam, lr_a, T = 0.1, 42, 1e-4, 0.1, 0.0
    w_r, phi_r, b_r = np.zeros(d, np.float32), np.zeros(d, np.float32), 0.0
    w, phi, b = dev(w_r), dev(phi_r), scalar_dev(0.0)
    yd, Tt = dev(y), scalar_dev(T)
    for t in range(2):
        idx = perm[t * P:(t + 1) * P]
        lr = float(np.float32(1.0 / np.sqrt(t + 1)))
        w_prev, phi_prev, b_prev = w_r, phi_r, b_r
        # the scores do not depend on the Philox key: take the first key under which no draw of
        # this pool falls into the rounding band of its keep probability
        for seed in range(42, 74):
            out = ref.step(Fh, y, idx, P, w_r, phi_r, b_r, gamma, seed, t, lam, lr, T, lr_a)
            if clear_draws(ref, out["prob"], gamma, seed, t).all():
                break
        else:
            pytest.fail("no Philox key with every draw clear of the rounding band")
        w_r, phi_r, b_r = out["w"], out["phi"], out["bias"]
        m = out["m"]
        cfg = api.step_config(gamma, lam, lr, lr_a, 0.0, seed, t, Tt)
        prob = torch.zeros(P, device="cuda")
        keep = torch.zeros(P, dtype=torch.uint8, device="cuda")
        pos = torch.zeros(P, dtype=torch.int32, device="cuda")
        ids = torch.zeros(P, dtype=torch.int32, device="cuda")
        loss = torch.zeros(P, device="cuda")
        cnt = torch.zeros(1, dtype=torch.int32, device="cuda")
        api.fused_step(F, yd, dev(idx), P, w, phi, b, cfg, None, prob, keep, pos, ids, loss, cnt, ws)
        assert int(host(cnt)[0]) == m
        assert np.array_equal(host(keep), out["keep"])
        assert np.array_equal(host(ids)[:m], out["kept_ids"])
        kept = out["kept_ids"]
        S = abs_dot_scale(Fh, kept, w_prev) + 1e-3
        assert_close_scaled(host(loss)[:m], out["loss"], S, f"loss step {t}")
        dots = _dots(Fh, kept, w_prev) * y[kept]
        on_kink = np.abs(dots - 1) <= RTOL * S
        absx_a = _col_abs_sum(Fh, kept[dots < 1], d)
        assert_close_scaled(host(w), w_r, np.abs(w_prev.astype(np.float64)) + lr / m * absx_a,
                            f"w step {t}", atol=lr / m * _col_abs_sum(Fh, kept[on_kink], d))
        absx = _col_abs_sum(Fh, kept, d)
        assert_close_scaled(host(phi), phi_r, np.abs(phi_prev.astype(np.float64)) + lr_a / m * absx,
                            f"phi step {t}")
        # the same step twice more from the same state: the same bits
        got = (host(w).copy(), host(phi).copy(), host(b).copy())
        for _ in range(2):
            w, phi, b = dev(w_prev), dev(phi_prev), scalar_dev(b_prev)
            api.fused_step(F, yd, dev(idx), P, w, phi, b, cfg, None, prob, keep, pos, ids, loss, cnt, ws)
            assert np.array_equal(host(w), got[0]) and np.array_equal(host(phi), got[1])
            assert np.array_equal(host(b), got[2])
        # the GPU state goes on from the oracle's bits so that step 2 is compared on equal inputs
        w, phi, b = dev(w_r), dev(phi_r), scalar_dev(b_r)


def test_train_epoch_on_csr_rows(ref, ws, sparse):
    """aa_train_epoch over CSR rows (general kernels) with the step-size schedule on the device:
    every step against the oracle step from the GPU's previous state at the single-step
    tolerances, then the epoch in one call bit for bit (tests/stepwise.py) -- and again, twice:
    the gradient sums do not depend on the order in which waves and blocks arrive."""
    from stepwise import check_epoch, run_whole
    rowptr, col, val, y, d = sparse
    n, P = 9000, 2048
    perm = rng(21).permutation(rowptr.size - 1)[:n].astype(np.int32)
    Fh = ref.Features.csr(rowptr, col, val, d)
    F = csr_features(rowptr, col, val, d)
    zeros = np.zeros(d, np.float32)
    args = dict(gamma=0.1, seed=42, step0=3, lam=1e-4, lr0=2.0, lr_a=0.3, T=0.0, ws=ws)
    counts, state = check_epoch(ref, Fh, F, y, perm, n, P, zeros, zeros, 0.0, **args)
    assert len(counts) == 5 and all(0 < m < P for m in counts) and state[3] == 5
    for _ in range(2):
        hist, _, _, again = run_whole(F, y, perm, n, P, zeros, zeros, 0.0, **args)
        assert hist == counts and again[3] == state[3]
        assert np.array_equal(again[0], state[0]) and np.array_equal(again[1], state[1])
        assert np.array_equal(again[2], state[2])
    # a constant step size (no counter) is still there
    w, phi, b = dev(zeros), dev(zeros), scalar_dev(0.0)
    Tt = scalar_dev(0.0)
    cfg = api.step_config(0.1, 1e-4, 0.5, 0.3, 0.0, 42, 3, Tt)
    hist = torch.full((5,), -1, dtype=torch.int32, device="cuda")
    api.train_epoch(F, dev(y), dev(perm), n, P, w, phi, b, cfg, None, hist, ws)
    assert host(hist).tolist()[0] == counts[0] and np.abs(host(w)).max() > 0


def _uniform_csr(r, n, d, nnz_lo, nnz_hi):
    """Rows whose columns are uniform over all of d (no hot columns), unit L2 norm."""
    lens = r.integers(nnz_lo, nnz_hi + 1, size=n)
    rowptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(lens, out=rowptr[1:])
    col = r.integers(0, d, size=int(rowptr[-1])).astype(np.int32)
    val = r.standard_normal(col.size).astype(np.float32)
    norm = np.sqrt(np.add.reduceat(val.astype(np.float64) ** 2, rowptr[:-1]))
    val = (val / np.repeat(norm, lens)).astype(np.float32)
    return rowptr, col, val


def _col_abs_sum_sp(Fh, ids, d):
    S = sp.csr_matrix((np.abs(Fh.val.astype(np.float64)), Fh.col, Fh.rowptr), shape=(Fh.n, d))
    return np.asarray(S[np.asarray(ids)].sum(axis=0)).ravel()


@pytest.mark.parametrize("n,nnz_lo,nnz_hi", [(300_000, 8, 16), (3000, 500, 700)])
def test_csr_updates_uniform_columns(ref, n, nnz_lo, nnz_hi):
    """Columns uniform over d = 2^18: nearly every entry falls outside the per-block table.
    300,000 short rows: every block makes two rounds, and most of its records are late ones.
    3000 rows of about 600 entries: the records of four rows per wave are more than a block's LDS,
    the bins and its late room hold (84 per candidate), so the excess goes to the accumulators."""
    r = rng(21)
    d, m = 1 << 18, n
    rowptr, col, val = _uniform_csr(r, n, d, nnz_lo, nnz_hi)
    y = np.where(r.random(n) < 0.5, -1.0, 1.0).astype(np.float32)
    w0 = (2.0 * r.standard_normal(d)).astype(np.float32)
    phi0 = r.standard_normal(d).astype(np.float32)
    rows = r.permutation(n)[:m].astype(np.int32)
    Fh = ref.Features.csr(rowptr, col, val, d)
    F = csr_features(rowptr, col, val, d)
    ws = api.Workspace(m, d)
    lam, lr, T, lr_a, b0 = 1e-3, 50.0, 0.8, 40.0, 0.1
    w_ref, loss_ref = ref.svm_sgd_step(Fh, y, rows, m, w0, lam, lr)
    S = abs_dot_scale(Fh, rows, w0)
    dots = _dots(Fh, rows, w0) * y[rows]
    on_kink = np.abs(dots - 1) <= RTOL * S
    assert on_kink.sum() <= 20
    w = dev(w0)
    loss = torch.zeros(m, device="cuda")
    api.svm_sgd_step(F, dev(y), dev(rows), scalar_dev(m, torch.int32), m, w, lam, lr, 0.0, loss, ws)
    assert_close_scaled(host(loss), loss_ref, S, "loss")
    absx = _col_abs_sum_sp(Fh, rows[dots < 1], d)
    assert_close_scaled(host(w), w_ref, np.abs(w0.astype(np.float64)) + lr / m * absx, "w",
                        atol=lr / m * _col_abs_sum_sp(Fh, rows[on_kink], d))
    assert np.abs(w_ref - w0).max() > 1e-3  # the step is visible at the tolerance
    w_bits = host(w).copy()
    for _ in range(2):   # (accumulators included: the same bits on every run)
        w = dev(w0)
        api.svm_sgd_step(F, dev(y), dev(rows), scalar_dev(m, torch.int32), m, w, lam, lr, 0.0, loss, ws)
        assert np.array_equal(host(w), w_bits)
    phi_ref, b_ref = ref.assistant_update(Fh, rows, m, loss_ref, T, phi0, b0, lr_a)
    phi, b = dev(phi0), scalar_dev(b0)
    api.assistant_update(F, dev(rows), scalar_dev(m, torch.int32), m, dev(loss_ref), scalar_dev(T),
                         phi, b, lr_a, 0.0, ws)
    absx = _col_abs_sum_sp(Fh, rows, d)
    assert_close_scaled(host(phi), phi_ref, np.abs(phi0.astype(np.float64)) + lr_a / m * absx, "phi")
    assert np.abs(phi_ref - phi0).max() > 2e-4  # 20 times the tolerance
    assert abs(float(host(b)[0]) - b_ref) <= RTOL * (abs(b0) + lr_a)


def test_train_epoch_with_overflowing_bins(ref):
    """aa_train_epoch over rows of about 600 entries with columns uniform over d = 2^18: in every
    step the records overflow LDS, the bins and the late room into the accumulators.  One step per call
    (each call prepares the workspace itself) is held to the oracle step at the single-step
    tolerances; then the epoch in one call, where from the second step on no launch prepares
    the workspace -- the update kernel of the step before has cleared what it read and has
    written the model pairs -- must give the same bits: a count or an accumulator left over, or
    a stale pair, would show.  Twice."""
    from stepwise import check_epoch, run_whole
    r = rng(33)
    n, d, P = 3000, 1 << 18, 1000
    rowptr, col, val = _uniform_csr(r, n, d, 500, 700)
    y = np.where(r.random(n) < 0.5, -1.0, 1.0).astype(np.float32)
    perm = r.permutation(n).astype(np.int32)
    Fh = ref.Features.csr(rowptr, col, val, d)
    F = csr_features(rowptr, col, val, d)
    ws = api.Workspace(P, d)
    w0 = (0.5 * r.standard_normal(d)).astype(np.float32)
    phi0 = (0.5 * r.standard_normal(d)).astype(np.float32)
    args = dict(gamma=0.3, seed=7, step0=0, lam=1e-3, lr0=20.0, lr_a=10.0, T=0.5, ws=ws)
    counts, state = check_epoch(ref, Fh, F, y, perm, n, P, w0, phi0, 0.1, **args)
    assert len(counts) == 3 and all(P // 4 < m <= P for m in counts)
    for _ in range(2):
        hist, _, _, again = run_whole(F, y, perm, n, P, w0, phi0, 0.1, **args)
        assert hist == counts
        assert np.array_equal(again[0], state[0]) and np.array_equal(again[1], state[1])
        assert np.array_equal(again[2], state[2])


def test_csr_fused_step_more_columns_than_the_bins_cover(ref):
    """d = 1,300,000 with both vectors updated: too many columns for the column bins, so every
    entry outside the per-block table goes to the dense accumulators."""
    r = rng(22)
    n, d, P = 6000, 1_300_000, 5000
    rowptr, col, val = _uniform_csr(r, n, d, 20, 40)
    y = np.where(r.random(n) < 0.5, -1.0, 1.0).astype(np.float32)
    w0 = (2.0 * r.standard_normal(d)).astype(np.float32)
    phi0 = (2.0 * r.standard_normal(d)).astype(np.float32)
    idx = r.permutation(n)[:P].astype(np.int32)
    Fh = ref.Features.csr(rowptr, col, val, d)
    F = csr_features(rowptr, col, val, d)
    ws = api.Workspace(P, d)
    b0, gamma, step, lam, lr, T, lr_a = 0.0, 0.1, 3, 1e-3, 0.5, 0.1, 0.3
    for seed in range(1, 20):
        out = ref.step(Fh, y, idx, P, w0, phi0, b0, gamma, seed, step, lam, lr, T, lr_a)
        if clear_draws(ref, out["prob"], gamma, seed, step).all():
            break
    else:
        raise AssertionError("no clear seed")
    kept = out["kept_ids"]
    dots = _dots(Fh, kept, w0) * y[kept]
    on_kink = np.abs(dots - 1) <= RTOL * abs_dot_scale(Fh, kept, w0)
    assert on_kink.sum() <= 3
    w, phi, b = dev(w0), dev(phi0), scalar_dev(b0)
    Tt = scalar_dev(T)
    cfg = api.step_config(gamma, lam, lr, lr_a, 0.0, seed, step, Tt)
    prob = torch.zeros(P, device="cuda")
    keep = torch.zeros(P, dtype=torch.uint8, device="cuda")
    pos = torch.zeros(P, dtype=torch.int32, device="cuda")
    ids = torch.zeros(P, dtype=torch.int32, device="cuda")
    loss = torch.zeros(P, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int32, device="cuda")
    api.fused_step(F, dev(y), dev(idx), P, w, phi, b, cfg, None, prob, keep, pos, ids, loss, cnt, ws)
    m = out["m"]
    assert int(host(cnt)[0]) == m
    assert np.array_equal(host(keep), out["keep"])
    assert np.array_equal(host(ids)[:m], out["kept_ids"])
    absx_a = _col_abs_sum_sp(Fh, kept[dots < 1], d)
    assert_close_scaled(host(w), out["w"], np.abs(w0.astype(np.float64)) + lr / m * absx_a, "w",
                        atol=lr / m * _col_abs_sum_sp(Fh, kept[on_kink], d))
    absx = _col_abs_sum_sp(Fh, kept, d)
    assert_close_scaled(host(phi), out["phi"], np.abs(phi0.astype(np.float64)) + lr_a / m * absx,
                        "phi")


def _workspace_counts(ws, table):
    """Table 0 (bins that left records in the blocks' late room), 1 (late records of a block) or 2 (bins whose accumulators
    were used) of the last pass: 256 integers each behind the 16 scalars that open the general kernels' part of the workspace."""
    first = ws.ptr - ws.buf.data_ptr() + 256 + 2 * 4 * 1024 + 256 + 4 * (16 + 256 * table)
    return host(ws.buf[first:first + 4 * 256]).view(np.int32)


def _late_records(ws):
    return _workspace_counts(ws, 1)


def _bins_with_accumulators(ws):
    """Bins of the last pass of which an entry found no room as a record."""
    return int(np.count_nonzero(_workspace_counts(ws, 2)))


def _check_csr_updates(ref, r, d, n, kind, lo, hi, with_val, misalign=False, all_rows=False, late=(0, 0)):
    """Boss step, Assistant update and both in one pass on random CSR rows of `lo` to `hi`
    entries against the oracle (columns uniform, Zipf-like, hot at the end of the range, or every 512 columns).
    misalign: the model vectors start 4 bytes past a 16-byte boundary.  all_rows: every row is chosen (a random
    number of them otherwise).  late: a block of the pass over one vector (all rows contribute) / over two has
    more late records than this."""
    def model(a):  # device copy of a model vector
        if not misalign:
            return dev(a)
        t = dev(np.concatenate([np.zeros(1, np.float32), a]))[1:]
        assert t.data_ptr() % 16 == 4
        return t
    lens = r.integers(lo, hi + 1, size=n)
    if r.random() < 0.2 and n > 1:
        lens[r.integers(1, n, size=max(1, n // 10))] = 0  # empty rows
    rowptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(lens, out=rowptr[1:])
    nnz = int(rowptr[-1])
    if kind == "uniform":
        col = r.integers(0, d, size=nnz)
    elif kind == "zipf":
        col = np.minimum(r.pareto(1.1, size=nnz).astype(np.int64), d - 1)
    elif kind == "fields":  # fields of 512 columns, each with a default in half of its entries
        col = 512 * r.integers(0, d // 512, size=nnz) + np.where(r.random(nnz) < 0.5, 0, r.integers(0, 512, size=nnz))
    elif kind == "one_bin":  # half of the entries on 200 columns of one bin (groups of four, 256 bins, see BinPlan)
        g = np.arange((d - 8192) // 4)
        mine = 8192 + 4 * g[(g + 157 * (g >> 8)) % 256 == 7]
        col = np.where(r.random(nnz) < 0.5, r.choice(mine, size=nnz) + r.integers(0, 4, size=nnz),
                       r.integers(0, d, size=nnz))
    else:  # a few very hot columns at the end of the range
        col = np.where(r.random(nnz) < 0.5, d - 1 - r.integers(0, min(3, d), size=nnz),
                       r.integers(0, d, size=nnz))
    col = col.astype(np.int32)
    val = r.standard_normal(nnz).astype(np.float32) if with_val else None
    y = np.where(r.random(n) < 0.5, -1.0, 1.0).astype(np.float32)
    w0 = (0.3 * r.standard_normal(d)).astype(np.float32)
    phi0 = (0.3 * r.standard_normal(d)).astype(np.float32)
    m = int(r.integers(1, n + 1))
    m = n if all_rows else m
    rows = r.permutation(n)[:m].astype(np.int32)
    tag = f"d={d} n={n} m={m} nnz={nnz} {kind}"
    Fh = ref.Features.csr(rowptr, col, val, d)
    F = csr_features(rowptr, col, val, d)
    ws = api.Workspace(m, d)
    vv = np.ones(nnz) if val is None else val.astype(np.float64)
    S = sp.csr_matrix((vv, col, rowptr), shape=(n, d))
    Sa = sp.csr_matrix((np.abs(vv), col, rowptr), shape=(n, d))
    lam, lr, T, lr_a, b0 = 1e-3, 0.7, 0.4, 0.5, 0.1
    w_ref, loss_ref = ref.svm_sgd_step(Fh, y, rows, m, w0, lam, lr)
    dots = (S[rows] @ w0.astype(np.float64)) * y[rows]
    Sdot = Sa[rows] @ np.abs(w0.astype(np.float64))
    kink = np.abs(dots - 1) <= RTOL * Sdot
    w = model(w0)
    loss = torch.zeros(m, device="cuda")
    api.svm_sgd_step(F, dev(y), dev(rows), scalar_dev(m, torch.int32), m, w, lam, lr, 0.0, loss, ws)
    assert_close_scaled(host(loss), loss_ref, Sdot, "loss " + tag, atol=1e-6)
    absx_w = np.asarray(Sa[rows[dots < 1]].sum(axis=0)).ravel()
    akink = np.asarray(Sa[rows[kink]].sum(axis=0)).ravel()
    assert_close_scaled(host(w), w_ref, np.abs(w0.astype(np.float64)) + lr / m * absx_w, "w " + tag,
                        atol=lr / m * akink)
    phi_ref, b_ref = ref.assistant_update(Fh, rows, m, loss_ref, T, phi0, b0, lr_a)
    phi, b = model(phi0), scalar_dev(b0)
    api.assistant_update(F, dev(rows), scalar_dev(m, torch.int32), m, dev(loss_ref),
                         scalar_dev(T), phi, b, lr_a, 0.0, ws)
    assert not late[0] or _late_records(ws).max() > late[0], tag
    absx = np.asarray(Sa[rows].sum(axis=0)).ravel()
    assert_close_scaled(host(phi), phi_ref, np.abs(phi0.astype(np.float64)) + lr_a / m * absx,
                        "phi " + tag)
    assert abs(float(host(b)[0]) - b_ref) <= RTOL * (abs(b0) + lr_a), tag
    # both updates in one pass over the rows (labels from the kernel's own losses: a row
    # whose loss sits within rounding of T may take either label)
    w, phi, b = model(w0), model(phi0), scalar_dev(b0)
    Tt = scalar_dev(T)
    cfg = api.step_config(0.0, lam, lr, lr_a, 0.0, 1, 0, Tt)
    api.boss_assistant_step(F, dev(y), dev(rows), scalar_dev(m, torch.int32), m, w, phi, b, cfg,
                            loss, ws)
    assert not late[1] or _late_records(ws).max() > late[1], tag
    assert_close_scaled(host(w), w_ref, np.abs(w0.astype(np.float64)) + lr / m * absx_w,
                        "w (one pass) " + tag, atol=lr / m * akink)
    on_T = np.abs(loss_ref.astype(np.float64) - T) <= RTOL * Sdot
    a_T = np.asarray(Sa[rows[on_T]].sum(axis=0)).ravel()
    assert_close_scaled(host(phi), phi_ref, np.abs(phi0.astype(np.float64)) + lr_a / m * absx,
                        "phi (one pass) " + tag, atol=lr_a / m * a_T)
    assert abs(float(host(b)[0]) - b_ref) <= RTOL * (abs(b0) + lr_a) + lr_a / m * on_T.sum(), tag


@pytest.mark.parametrize("block", range(4))
def test_csr_updates_random_shapes(ref, block):
    """Randomised shapes for the CSR Boss step and Assistant update: d from 37 to 1,200,000
    (below, at and above the sizes of the per-block LDS table, and beyond what the column bins
    cover), 1 to 40,000 rows of 0 to 200 entries, uniform / Zipf-like / hot-at-the-end columns,
    with and without values."""
    master = rng(7000 + block)
    for case in range(6):
        r = rng(int(master.integers(1 << 30)))
        d = int(r.choice([37, 600, 3072, 4096, 5000, 8192, 8193, 20000, 70000, 300000, 1 << 20, 1_200_000]))
        n = int(r.choice([1, 7, 300, 5000, 40000]))
        kind = r.choice(["uniform", "zipf", "hot_tail"])
        lo, hi = (1, 12) if r.random() < 0.5 else (30, 200)
        n = min(n, 3_000_000 // hi)
        _check_csr_updates(ref, r, d, n, kind, lo, hi, r.random() >= 0.3)


def test_csr_updates_with_model_vectors_off_16_byte_alignment(ref):
    """The bin owners move four model columns per 128-bit access wherever the vectors start."""
    r = rng(77)
    _check_csr_updates(ref, r, 20001, 3000, "zipf", 20, 60, True, misalign=True)
    _check_csr_updates(ref, r, 300000, 3000, "hot_tail", 20, 60, False, misalign=True)


@pytest.mark.parametrize("d", [1, 3, 3071, 3072, 8191, 8192])
def test_csr_updates_whose_columns_are_all_in_the_table(ref, d):
    """3072 columns of a pass over two vectors, 8192 of one over one, have their own slots: no tags, records and gathers."""
    r = rng(700 + d)
    _check_csr_updates(ref, r, d, 2000, "hot_tail", 0, 70, True)
    _check_csr_updates(ref, r, d, 300, "uniform", 120, 140, False)


@pytest.mark.parametrize("d", [3073, 3075, 3079, 3072 + 1021, 8193, 8195, 8192 + 1022,
                               3072 + (1 << 18), 3072 + (1 << 18) + 5, 8192 + (1 << 18), 8192 + (1 << 18) + 6])
def test_csr_updates_at_the_edges_of_the_column_bins(ref, d):
    """Feature counts just past the per-block table (3072 columns when both vectors are
    updated, 8192 with one): one, three, seven columns for the bins, a count that is no
    multiple of four (the owners fold four neighbours at a time and finish the model's last
    columns singly), fewer groups than bins, and both sides of the count at which the bins
    change from groups of 4 to groups of 16 columns.  Hot columns at the end of the range."""
    r = rng(900 + d % 1000)
    _check_csr_updates(ref, r, d, 2000, "hot_tail", 20, 60, True)
    _check_csr_updates(ref, r, d, 300, "uniform", 1, 12, False)


@pytest.mark.parametrize("n,d,kind,lo,hi,with_val,late", [
    (40_000, 60_000, "uniform", 40, 90, True, (4000, 2000)),      # two rows a unit and rows of their own
    (40_000, 9000, "hot_tail", 0, 5, False, (0, 0)),              # empty rows, and some before the matrix's fourth entry
    (40_000, 4000, "zipf", 63, 65, True, (0, 0)),                 # both sides of one piece of 64 entries
    (30_000, 70_000, "hot_tail", 127, 129, False, (0, 0)),        # both sides of two
    (20_000, 300_000, "uniform", 100, 200, True, (1000, 400)),    # rows past two pieces, no late room left
    (64, 200_000, "uniform", 380, 420, True, (16_384, 12_288)),   # one block, several sorted pieces
    (110_000, 300_000, "uniform", 42, 46, True, (0, 12_288)),     # 256 blocks, two sorted pieces
    (40_000, 60_000, "one_bin", 40, 70, True, (2000, 1000))])     # late records of which one bin takes only the first
def test_csr_updates_pieces_pairs_and_late_records(ref, n, d, kind, lo, hi, with_val, late):
    """All rows chosen.  30,000 rows are at least seven a wave, more than it has lane groups: short rows go two to a unit.
    Records beyond a block's LDS are late ones, sorted by bin in pieces of at most 16,384 (one vector) and 12,288 (two)."""
    _check_csr_updates(ref, rng(n + d), d, n, kind, lo, hi, with_val, all_rows=True, late=late)


@pytest.mark.parametrize("d", [TABLE_MIN_COLS + 1, TABLE_MIN_COLS + 3, TABLE_COLS - 1, TABLE_COLS, TABLE_COLS + 1, 64_002])
@pytest.mark.parametrize("with_val", [True, False])
def test_csr_scores_with_the_table_and_without(d, with_val):
    """The fewest rows that are scored with phi's first entries in LDS, and one row less, without.  The
    order of additions is the same: the same bits, whether the table ends with the model, between its fours or before it."""
    n, r = TABLE_ROWS, rng(d)
    lens = r.integers(0, 140, size=n)
    rowptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(lens, out=rowptr[1:])
    nnz = int(rowptr[-1])
    col = np.where(r.random(nnz) < 0.2, d - 1 - r.integers(0, 5, size=nnz), r.integers(0, d, size=nnz)).astype(np.int32)
    F = csr_features(rowptr, col, r.standard_normal(nnz).astype(np.float32) if with_val else None, d)
    phi, b = dev((0.1 * r.standard_normal(d + 1)).astype(np.float32))[1:], scalar_dev(0.1)
    rows = dev(r.permutation(n).astype(np.int32))
    with_table, without = torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")
    api.assistant_score(F, rows, n, phi, b, None, with_table)
    api.assistant_score(F, rows, n - 1, phi, b, None, without)
    assert torch.equal(with_table[:-1], without[:-1]) and float(with_table[-1]) > 0.0


@pytest.mark.parametrize("d", [80 * 512, 20 * 512])
def test_csr_updates_frequent_columns_512_apart(ref, d):
    """Fields padded to 512 columns, each with a frequent default: columns 512, 1024, 2048 ... apart past the table
    compete for the hashed slots."""
    _check_csr_updates(ref, rng(512 + d), d, 6000, "fields", 40, 100, True)


def test_csr_frequent_columns_a_power_of_two_apart_take_no_longer():
    """A whole step over rows of 80 fields takes about as long with fields of 512 or 1024 columns as with fields of 1000 (3.6
    and 2.2 times when frequent columns a power of two apart lost their hashed slots to each other in every
    block; 1.3 and 1.6 times when the records of their slots all met in two bins or one)."""
    n, fields = 65_536, 80
    r = rng(61)
    field, other = np.arange(n * fields) % fields, r.random(n * fields)
    default = r.random(n * fields) < 0.5
    val = (r.standard_normal(n * fields) / 9.0).astype(np.float32)
    y, idx = dev(np.where(r.random(n) < 0.5, -1.0, 1.0).astype(np.float32)), dev(r.permutation(n).astype(np.int32))
    cfg = api.step_config(0.1, 0.0, 1e-7, 1e-7, 0.0, 3, 1, scalar_dev(0.5))
    times = {}
    for width in (512, 1024, 1000):
        d = fields * width
        col = (field * width + np.where(default, 0, (other * width).astype(np.int64))).astype(np.int32)
        F = csr_features(np.arange(0, n * fields + 1, fields, dtype=np.int64), col, val, d)
        w, phi, b = (dev((0.1 * r.standard_normal(k)).astype(np.float32)) for k in (d, d, 1))
        ws = api.Workspace(n, d)
        prob, loss = torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")
        keep = torch.zeros(n, dtype=torch.uint8, device="cuda")
        pos, ids, cnt = (torch.zeros(k, dtype=torch.int32, device="cuda") for k in (n, n, 1))
        times[width] = _device_time(lambda: api.fused_step(F, y, idx, n, w, phi, b, cfg, None, prob, keep, pos, ids, loss,
                                                           cnt, ws))
    assert max(times[512], times[1024]) < 1.3 * times[1000], times


def test_csr_records_of_one_block_in_one_bin():
    """The rows of one block of the pass have all their columns in one column bin, far more than a block has hashed slots:
    its records are one run of thousands.  The sums are right, and the update takes about as long as with the
    same rows spread over all columns (twice to three times when sixteen lanes read such a run alone)."""
    n, d, per, few = 65_536, 1_500_000, 60, 2
    r = rng(67)
    lens = np.where(np.arange(n) < 256, per, few)
    rowptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(lens, out=rowptr[1:])
    nnz, head = int(rowptr[-1]), 256 * per
    spread = r.integers(8192, d, size=nnz)
    one_bin = spread.copy()
    one_bin[:head] = 8192 + 16 * 256 * r.integers(0, 360, size=head) + r.integers(0, 16, size=head)
    ws, loss, T = api.Workspace(n, d), torch.full((n,), 0.7, device="cuda"), scalar_dev(0.5)
    m, times = scalar_dev(n, torch.int32), {}
    for name, col in (("spread", spread), ("one bin", one_bin)):
        F = csr_features(rowptr, col.astype(np.int32), None, d)
        phi, b = torch.zeros(d, device="cuda"), scalar_dev(0.0)
        api.assistant_update(F, None, m, n, loss, T, phi, b, 1.0, 0.0, ws)
        # g = 1/2, z = 1: every entry moves its column by 1 / (2 n), exactly
        assert np.array_equal(host(phi), (np.bincount(col, minlength=d) / (2.0 * n)).astype(np.float32))
        times[name] = _device_time(lambda: api.assistant_update(F, None, m, n, loss, T, phi, b, 0.0, 0.0, ws))
    assert times["one bin"] < 1.5 * times["spread"], times


@pytest.mark.parametrize("kind", ["uniform", "fields"])
def test_csr_records_that_find_their_bin_full(ref, kind):
    """48 records a candidate, evenly spread: there is room for all of them; and fields of 512 columns, each with a frequent
    one.  A record whose bin is full joins its block's late
    ones: nothing is left to the atomics on the accumulators, and the sums are right."""
    r = rng(71)
    n, per, d = (16_384, 48, 60_000) if kind == "uniform" else (32_768, 40, 80 * 512)  # (1 / 2n is exact)
    if kind == "uniform":
        col = r.integers(8192, d, size=n * per)
    else:
        col = 512 * r.integers(16, 80, size=n * per) + np.where(r.random(n * per) < 0.5, 0, r.integers(0, 512, size=n * per))
    rowptr = np.arange(0, n * per + 1, per, dtype=np.int64)
    F, ws = csr_features(rowptr, col.astype(np.int32), None, d), api.Workspace(n, d)
    m, y, loss = scalar_dev(n, torch.int32), dev(np.ones(n, np.float32)), torch.full((n,), 0.7, device="cuda")
    want = (np.bincount(col, minlength=d) / (2.0 * n)).astype(np.float32)
    phi, b = torch.zeros(d, device="cuda"), scalar_dev(0.0)
    api.assistant_update(F, None, m, n, loss, scalar_dev(0.5), phi, b, 1.0, 0.0, ws)  # (g = 1/2, z = 1)
    assert _bins_with_accumulators(ws) == 0 and np.array_equal(host(phi), want)
    w = torch.zeros(d, device="cuda")
    phi.zero_()
    b.zero_()
    cfg = api.step_config(0.0, 0.0, 0.5, 1.0, 0.0, 1, 0, scalar_dev(0.5))
    api.boss_assistant_step(F, y, None, m, n, w, phi, b, cfg, loss, ws)               # (margin 0, loss 1)
    assert _bins_with_accumulators(ws) == 0
    assert np.array_equal(host(phi), want) and np.array_equal(host(w), want)


def _exact_updates(n, d, rowptr, col, two):
    """One update (g = 1/2 and z = 1, with margin 0 and loss 1) of an Assistant, or of both vectors, that moves a column by 1 /
    (2 n) for every entry, exactly; returns the workspace."""
    F, ws = csr_features(rowptr, col, None, d), api.Workspace(n, d)
    m, y, loss = scalar_dev(n, torch.int32), dev(np.ones(n, np.float32)), torch.full((n,), 0.7, device="cuda")
    phi, w, b = torch.zeros(d, device="cuda"), torch.zeros(d, device="cuda"), scalar_dev(0.0)
    if two:
        cfg = api.step_config(0.0, 0.0, 0.5, 1.0, 0.0, 1, 0, scalar_dev(0.5))
        api.boss_assistant_step(F, y, None, m, n, w, phi, b, cfg, loss, ws)
    else:
        api.assistant_update(F, None, m, n, loss, scalar_dev(0.5), phi, b, 1.0, 0.0, ws)
    want = (np.bincount(col, minlength=d) / (2.0 * n)).astype(np.float32)
    assert np.array_equal(host(phi), want) and (not two or np.array_equal(host(w), want))
    return ws


@pytest.mark.parametrize("two,per", [(False, 78), (True, 52)])
def test_csr_room_for_the_late_records_of_a_large_pool(two, per):
    """Of 84 records a candidate (56 of both vectors) the blocks of a large pool can place nearly all while they walk their
    rows, whatever the bins have room for meanwhile: rows of 78 (52) columns that are not in the table leave nothing to the
    accumulators."""
    n, d = 1 << 18, 500_000
    col = rng(79).integers(8192, d, size=n * per, dtype=np.int32)
    ws = _exact_updates(n, d, np.arange(0, n * per + 1, per, dtype=np.int64), col, two)
    assert _bins_with_accumulators(ws) == 0 and _late_records(ws).min() > (per - 10) * n // 256 - 6000


@pytest.mark.parametrize("two", [False, True])
@pytest.mark.parametrize("first,second", [("long", "long"), ("long", "short"), ("short", "short")])
def test_csr_late_records_stay_or_go_to_the_bins(two, first, second):
    """Blocks with more late records than their share of the bins has room for leave all of them in their pieces, others none:
    all blocks, half of them, and none, in the first and the second half of the rows."""
    n, d = 65_536, 300_000
    lens = {"long": 49 if two else 70, "short": 28 if two else 34}  # (a block has 256 rows, and room for 13,056 or 20,480 records)
    rowptr = np.r_[0, np.cumsum(np.repeat([lens[first], lens[second]], n // 2))]
    col = rng(83).integers(8192, d, size=int(rowptr[-1]), dtype=np.int32)
    ws = _exact_updates(n, d, rowptr, col, two)
    late, left = _late_records(ws), int(np.count_nonzero(_workspace_counts(ws, 0)))
    assert late.min() > 0 and (late[:128] > 2 * late[128:]).all() == (first != second)
    assert _bins_with_accumulators(ws) == 0 and left == (256 if first == "long" else 0)


@pytest.mark.parametrize("ones", [True, False])
def test_csr_rows_past_two_to_the_29_entries(ref, ones):
    """Rows on both sides of entry 2^29, where 32-bit byte offsets end, behind a row of half a thousand million entries that is
    not chosen: scores (general kernel; with many pool places over these columns the one with phi in LDS) and updates have
    the bits of the same rows in a matrix of their own, and the oracle's values."""
    r = rng(73)
    n, d = 400, 20_000
    assert TABLE_MIN_COLS < d <= 2 * TABLE_COLS
    lens = np.where(r.random(n) < 0.5, r.integers(0, 70, size=n), r.integers(60, 300, size=n))
    own = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(lens, out=own[1:])
    nnz, skipped = int(own[-1]), (1 << 29) - int(own[n // 2]) - 3
    col = r.integers(0, d, size=nnz).astype(np.int32)
    val = None if ones else (r.standard_normal(nnz) / 8.0).astype(np.float32)
    far_col = torch.zeros(skipped + nnz, dtype=torch.int32, device="cuda")
    far_col[skipped:] = dev(col)
    far_val = None
    if not ones:
        far_val = torch.zeros(skipped + nnz, dtype=torch.float32, device="cuda")
        far_val[skipped:] = dev(val)
    near = csr_features(own, col, val, d)
    far = api.Features.csr(dev(np.r_[0, own + skipped]), far_col, far_val, d)  # (row k + 1 is the other's row k)
    phi0 = (r.standard_normal(d) / 8.0).astype(np.float32)
    w0 = (r.standard_normal(d) / 8.0).astype(np.float32)
    y = np.where(r.random(n) < 0.5, -1.0, 1.0).astype(np.float32)
    Fh = ref.Features.csr(own, col, val, d)
    ws, got = api.Workspace(n, d), {}
    for name, F, shift in (("near", near, 0), ("far", far, 1)):
        out = []
        for P in (n, TABLE_ROWS):
            ids = dev((np.arange(P) % n + shift).astype(np.int32))
            out += [torch.zeros(P, device="cuda"), torch.zeros(P, device="cuda")]
            api.assistant_score(F, ids, P, dev(phi0), scalar_dev(0.1), out[-2], out[-1])
        ids, m = dev((np.arange(n) + shift).astype(np.int32)), scalar_dev(n, torch.int32)
        yd = dev(np.r_[np.zeros(shift, np.float32), y])
        w, phi, b, loss = dev(w0), dev(phi0), scalar_dev(0.1), torch.zeros(n, device="cuda")
        cfg = api.step_config(0.0, 1e-3, 0.7, 0.5, 0.0, 1, 0, scalar_dev(0.4))
        api.boss_assistant_step(F, yd, ids, m, n, w, phi, b, cfg, loss, ws)
        w1 = dev(w0)
        api.svm_sgd_step(F, yd, ids, m, n, w1, 1e-3, 0.7, 0.0, loss, ws)
        got[name] = [host(t).copy() for t in out + [w, phi, b, loss, w1]]
    for x, z in zip(got["near"], got["far"]):
        assert np.array_equal(x, z)
    ref_logit, ref_prob = ref.assistant_score(Fh, None, n, phi0, bias=0.1)
    assert_logit_prob(got["far"][0], got["far"][1], ref_logit, ref_prob, abs_dot_scale(Fh, np.arange(n), phi0), bias=0.1)
    assert np.array_equal(got["far"][2], np.resize(got["far"][0], TABLE_ROWS))
    w_ref, loss_ref = ref.svm_sgd_step(Fh, y, np.arange(n, dtype=np.int32), n, w0, 1e-3, 0.7)
    assert_close_scaled(got["far"][7], loss_ref, abs_dot_scale(Fh, np.arange(n), w0), "loss", atol=1e-6)
    scale = np.abs(w0.astype(np.float64)) + 0.7 / n * _col_abs_sum(Fh, np.arange(n), d)
    assert_close_scaled(got["far"][8], w_ref, scale, "w")


def test_csr_hashed_sum_beyond_float_range():
    """A column past the table whose sum no float holds, and one whose sum is no number: the column's total
    is rounded once (to an infinity, a NaN), and nothing else is touched by it."""
    n, d, big, nan = 64, 9000, 8999, 8995
    cols = np.stack([np.full(n, 5), np.full(n, nan), np.full(n, big)], axis=1).astype(np.int32)
    vals = np.stack([np.ones(n), np.ones(n), np.full(n, 3e38)], axis=1).astype(np.float32)
    vals[3, 1] = np.nan
    F = csr_features(np.arange(0, 3 * n + 1, 3, dtype=np.int64), cols.ravel(), vals.ravel(), d)
    phi, b = torch.zeros(d, device="cuda"), scalar_dev(0.0)
    keep = [i for i in range(n) if i != 3]
    ws = api.Workspace(n, d)
    api.assistant_update(F, dev(np.array(keep, np.int32)), scalar_dev(n - 1, torch.int32), n - 1,
                         torch.zeros(n - 1, device="cuda"), scalar_dev(1.0), phi, b, 1.0, 0.0, ws)
    got = host(phi)
    assert got[big] == -np.inf and np.isclose(got[5], -0.5) and np.isclose(got[nan], -0.5)
    assert np.count_nonzero(got) == 3 and np.isclose(float(host(b)[0]), -0.5)
    phi.zero_()
    api.assistant_update(F, None, scalar_dev(n, torch.int32), n, torch.zeros(n, device="cuda"), scalar_dev(1.0),
                         phi, b, 1.0, 0.0, ws)
    got = host(phi)
    assert np.isnan(got[[5, nan, big]]).all() and np.count_nonzero(got) == 3   # (row 3's residual is a NaN)
