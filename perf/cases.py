"""Cases the framework is timed on: what a program that uses it has it do, over the sizes it is used at.

A case is a dict of plain values; its "kind" says which calls a pass makes:

  step     one whole step on one pool of dense rows (fused_step)
  epoch    one epoch of whole steps on dense rows (train_epoch); any row width
  staged   the same step as separate calls: score, shrink, gather of rows, labels and ids, Boss step,
           Assistant update -- what a program does whose Boss is not the linear SVM
  sk       one epoch of hard-threshold shrinking on dense rows (sk_epoch)
  stale    one epoch of the two-stream Boss / Assistant pipeline (train_epoch_stale)
  sparse   one epoch of whole steps on CSR rows (train_epoch)
  images   image batch generator: score + keep + compact, gather of the kept images, then per batch the
           running-median threshold and the Assistant update
  batches  translation batch generator: score + keep + compact of token lists, lengths of the kept pairs,
           length-bucketed batches, compacted CSR rows
  update   translation batch generator: the Assistant update over the kept pairs

Model state lives on as in a training program: a second pass goes on from where the first one ended.
All inputs are drawn on the GPU from the seed.
"""
import math

import torch

from paper_1905_03381_amd import api

GAMMA, LAM, LR_A, PHILOX = 0.1, 1e-4, 0.1, 42


def listed():
    return [
        # The smallest step in use (10,000 x 128 rows, pools of 256): two dependent launches, nothing else.
        {"name": "step_tiny", "kind": "step", "n": 10_000, "d": 128, "P": 256},
        # One epoch at that size in one call: forty steps that are all launch and latency.
        {"name": "epoch_tiny", "kind": "epoch", "n": 10_000, "d": 128, "P": 256},
        # The benchmark's step (d = 1024, pools of 16,384), seven pools and the short one an epoch ends with.
        {"name": "epoch_dense", "kind": "epoch", "n": 7 * 16_384 + 576, "d": 1024, "P": 16_384},
        # The largest pool the dense path is documented for per step: a launch that can fill the memory system.
        {"name": "step_dense_large", "kind": "step", "n": 300_000, "d": 1024, "P": 262_144},
        # Rows that do not fill the lane layout (d = 1000) and a ragged pool, through the separate calls.
        {"name": "staged_dense", "kind": "staged", "n": 60_000, "d": 1000, "P": 12_345},
        # Hard-threshold shrinking (no Assistant), half-width rows, ragged last pool.
        {"name": "sk_epoch", "kind": "sk", "n": 8 * 8192 + 1000, "d": 512, "P": 8192},
        # The asynchronous schedule: generator and Boss on two streams, two batches in the queue.
        {"name": "stale_epoch", "kind": "stale", "n": 5 * 16_384 + 576, "d": 1024, "P": 16_384, "staleness": 2},
        # Rows no register layout takes (odd, wider than 2048): the general kernels on dense rows.
        {"name": "epoch_wide_rows", "kind": "epoch", "n": 4 * 4096 + 77, "d": 4137, "P": 4096},
        # The sparse linear SVM: 2^20 columns, Zipf(1.1) column ids, about 100 entries a row, pools of 65,536.
        {"name": "sparse_epoch", "kind": "sparse", "n": 3 * 65_536 + 3392, "d": 1 << 20, "P": 65_536, "nnz": 100},
        # The image batch generator: 512 features a candidate, 3 x 224 x 224 byte images, batches of 256.
        {"name": "images", "kind": "images", "P": 8192, "d": 512, "row_bytes": 150_528, "B": 256},
        # The translation batch generator's assembly half, at its full size.
        {"name": "translation_batches", "kind": "batches", "n": 1_000_000, "vocab": 32_000, "ones": False},
        # And its learning half.
        {"name": "translation_update", "kind": "update", "n": 1_000_000, "vocab": 32_000, "ones": False},
    ]


def _log(rng, lo, hi):
    """A whole number from lo to hi, even over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["step", "step", "epoch", "epoch", "wide", "staged", "sk", "stale", "sparse", "sparse",
                       "images", "batches", "update"])
    if kind in ("step", "epoch", "staged", "sk", "stale"):
        # widths of the register layouts: full ones (256, 512, 1024, 2048) and any multiple of four
        d = rng.choice([256, 512, 1024, 2048]) if rng.random() < 0.4 else 4 * _log(rng, 9, 512)
        top = 262_144 if kind == "step" else 65_536 if kind == "epoch" else 20_000
        P = _log(rng, 100, min(top, (1 << 28) // d))
        steps = {"step": 1, "staged": 1, "stale": rng.randint(2, 5)}.get(kind, rng.randint(2, 6))
        n = (steps - 1) * P + rng.randint(1, P) if steps > 1 else P + rng.randint(0, P // 4)
        case = {"kind": kind, "n": n, "d": d, "P": P}
        if kind == "stale":
            case["staleness"] = rng.randint(0, 3)
        return case
    if kind == "wide":  # rows for the general kernels: wider than 2048, or not a multiple of four
        d = _log(rng, 2049, 8000) if rng.random() < 0.6 else _log(rng, 30, 2000) | 1
        P = _log(rng, 200, min(8192, (1 << 25) // d))
        return {"kind": "epoch", "n": 3 * P + rng.randint(1, P), "d": d, "P": P}
    if kind == "sparse":
        P = _log(rng, 1000, 65_536)
        return {"kind": "sparse", "n": rng.randint(1, 2) * P + rng.randint(1, P), "d": _log(rng, 1 << 13, 1 << 20),
                "P": P, "nnz": _log(rng, 10, 150)}
    if kind == "images":
        side = rng.choice([28, 32, 33, 64, 96, 128, 224])
        return {"kind": "images", "P": _log(rng, 600, 8192), "d": 4 * _log(rng, 16, 256),
                "row_bytes": 3 * side * side, "B": rng.choice([32, 64, 100, 128, 256, 512])}
    return {"kind": kind, "n": _log(rng, 5_000, 1_000_000), "vocab": _log(rng, 2_000, 32_000),
            "ones": rng.random() < 0.4}


# ---------------------------------------------------------------------------
# inputs


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 7919 + 13)
    return g


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda")


def _uniform(g, *shape):
    return torch.rand(*shape, generator=g, device="cuda")


def _perm(g, n):
    return torch.randperm(n, generator=g, device="cuda").to(torch.int32)


def _zeros(n, dtype=torch.float32):
    return torch.zeros(n, dtype=dtype, device="cuda")


def _dense(g, n, d):
    """Unit-norm Gaussian rows, labels from a planted vector with 5 % flips, a half-learnt Boss
    and an Assistant that is as yet undecided."""
    x = _normal(g, n, d)
    x /= x.norm(dim=1, keepdim=True)
    w_star = _normal(g, d) * math.sqrt(1024.0 / d)
    y = torch.where(x.double() @ w_star.double() >= 0, 1.0, -1.0).float()
    y = torch.where(_uniform(g, n) < 0.05, -y, y)
    w = 0.5 * w_star + _normal(g, d)
    return x, y, w, _normal(g, d) * math.sqrt(1.0 / 32), torch.full((1,), 0.2, device="cuda")


def _zipf(items, exponent):
    p = 1.0 / torch.arange(1, items + 1, dtype=torch.float64) ** exponent
    c = torch.cumsum(p, 0)
    return (c / c[-1]).cuda()


def _tokens(g, cdf, count):
    t = torch.searchsorted(cdf, torch.rand(count, generator=g, device="cuda", dtype=torch.float64))
    return t.clamp_(max=cdf.numel() - 1)


def _sparse_rows(g, n, d, mean_nnz):
    """CSR rows: max(1, Poisson) distinct Zipf(1.1) columns, ascending, lognormal values of unit norm."""
    want = torch.poisson(torch.full((n,), float(mean_nnz), device="cuda"), generator=g).long().clamp_(1, d // 2)
    draws = 2 * want + 16
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), draws)
    key = row * d + _tokens(g, _zipf(d, 1.1), row.numel())
    key, order = torch.sort(key, stable=True)            # the first draw of a column stands for it
    first = torch.ones_like(key, dtype=torch.bool)
    first[1:] = key[1:] != key[:-1]
    at, back = torch.sort(order[first])                  # the distinct ones in the order they were drawn
    key = key[first][back]
    row = key // d
    have = torch.bincount(row, minlength=n)
    start = torch.cumsum(have, 0) - have
    rank = torch.arange(key.numel(), device="cuda") - start[row]
    key = torch.sort(key[rank < want[row]])[0]
    row, col = key // d, (key % d).to(torch.int32)
    have = torch.bincount(row, minlength=n)
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rowptr[1:] = torch.cumsum(have, 0)
    val = torch.exp(_normal(g, key.numel()))
    norm = torch.segment_reduce((val * val).double(), "sum", lengths=have).sqrt().float()
    return rowptr, col, val / norm[row], row, have


def _pairs(g, n, vocab, ones):
    """Sentence pairs as token lists: source tokens, target tokens (ids after the source's) and,
    unless every entry is one, two length features."""
    extra = 0 if ones else 2
    ls, lt = (torch.poisson(torch.full((n,), 27.0, device="cuda"), generator=g).clamp_(1, 128).long() for _ in "st")
    have = ls + lt + extra
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rowptr[1:] = torch.cumsum(have, 0)
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), have)
    pos = torch.arange(row.numel(), device="cuda") - rowptr[row]
    col = _tokens(g, _zipf(vocab, 1.0), row.numel())
    a, b = ls[row], ls[row] + lt[row]
    col = torch.where(pos >= a, col + vocab, col)
    val = None
    if not ones:
        col = torch.where(pos >= b, 2 * vocab + (pos - b), col)
        val = torch.where(pos == b, ls[row] / 128.0, torch.where(pos > b, lt[row] / 128.0, 1.0)).float()
    return rowptr, col.to(torch.int32), val, ls.to(torch.int32), lt.to(torch.int32), 2 * vocab + extra


def _gamma2(g, n, scale):
    """Gamma(2, scale) losses: the sum of two exponentials."""
    return (-(torch.log1p(-_uniform(g, n)) + torch.log1p(-_uniform(g, n))) * scale).float()


def _config(lr, T, lr_a=LR_A):
    return api.step_config(GAMMA, LAM, lr, lr_a, 0.0, PHILOX, 0, T)


def prepare(case, seed):
    g, k = _gen(seed), case["kind"]
    s = {"case": case}
    if k in ("step", "epoch", "staged", "sk", "stale"):
        n, d, P = case["n"], case["d"], case["P"]
        s["x"], s["y"], s["w"], s["phi"], s["b"] = _dense(g, n, d)
        s["F"] = api.Features.dense(s["x"])
    elif k == "sparse":
        n, d, P = case["n"], case["d"], case["P"]
        rowptr, col, val, row, have = _sparse_rows(g, n, d, case["nnz"])
        w_star = torch.where(_uniform(g, d) < 0.01, _normal(g, d), 0.0)
        w_star[:64] = _normal(g, 64)
        score = torch.segment_reduce(val.double() * w_star.double()[col.long()], "sum", lengths=have)
        y = torch.where(score >= 0, 1.0, -1.0).float()
        s["y"] = torch.where(_uniform(g, n) < 0.05, -y, y)
        s["w"] = 0.5 * w_star + 0.5 * _normal(g, d)
        s["phi"], s["b"] = 0.5 * _normal(g, d), torch.full((1,), 0.2, device="cuda")
        s["F"] = api.Features.csr(rowptr, col, val, d)
        s["rows"] = (rowptr, col, val)
    if k in ("step", "staged"):
        s["ws"] = api.Workspace(P, d)
        s["idx"] = _perm(g, n)[:P].contiguous()
        s["T"] = torch.full((1,), 0.25, device="cuda")
        s["cfg"] = _config(8.0, s["T"])
        for name in ("prob", "loss"):
            s[name] = _zeros(P)
        s["keep"], s["cnt"] = _zeros(P, torch.uint8), _zeros(1, torch.int32)
        s["pos"], s["ids"] = _zeros(P, torch.int32), _zeros(P, torch.int32)
        if k == "staged":
            s["xk"], s["yk"] = _zeros(P * d).view(P, d), _zeros(P)
            s["Fk"] = api.Features.dense(s["xk"])
    elif k in ("epoch", "sk", "stale", "sparse"):
        stale = case.get("staleness")
        s["ws"] = api.Workspace(P, d, staleness=stale)
        s["perm"] = _perm(g, n)
        s["T"] = torch.full((1,), 0.5 if k in ("sparse", "sk") else 0.25, device="cuda")
        s["cfg"] = _config(4.0 if k == "sparse" else 32.0, s["T"])
        steps = -(-n // P)
        s["t"], s["hist"] = _zeros(1, torch.int32), _zeros(steps, torch.int32)
        s["ids"], s["loss"] = _zeros(steps * P, torch.int32), _zeros(steps * P)
        if k == "stale":
            s["side"] = torch.cuda.Stream()
    elif k == "images":
        P, d = case["P"], case["d"]
        s["x"] = _normal(g, P, d)
        s["F"], s["ws"] = api.Features.dense(s["x"]), api.Workspace(P, d)
        s["store"] = torch.randint(0, 256, (P, case["row_bytes"]), generator=g, device="cuda", dtype=torch.uint8)
        s["batches"] = torch.zeros_like(s["store"])
        s["phi"], s["b"] = _normal(g, d) / math.sqrt(d), _zeros(1)
        s["idx"], s["losses"] = _perm(g, P), _gamma2(g, P, 0.5)
        s["prob"], s["keep"] = _zeros(P), _zeros(P, torch.uint8)
        s["pos"], s["ids"], s["cnt"] = _zeros(P, torch.int32), _zeros(P, torch.int32), _zeros(1, torch.int32)
        s["T"], s["init"] = _zeros(1), _zeros(1, torch.int32)
        s["full"], s["rest"] = torch.full((1,), case["B"], dtype=torch.int32, device="cuda"), _zeros(1, torch.int32)
    elif k in ("batches", "update"):
        n = case["n"]
        rowptr, col, val, s["ls"], s["lt"], d = _pairs(g, n, case["vocab"], case["ones"])
        s["rows"], s["F"], s["ws"] = (rowptr, col, val), api.Features.csr(rowptr, col, val, d), api.Workspace(n, d)
        s["phi"], s["b"] = 0.05 * _normal(g, d), torch.full((1,), -0.2, device="cuda")
        s["pos"], s["cnt"] = _zeros(n, torch.int32), _zeros(1, torch.int32)
        if k == "batches":
            s["prob"], s["keep"] = _zeros(n), _zeros(n, torch.uint8)
            s["ls_k"], s["lt_k"], s["order"], s["batch_of"] = (_zeros(n, torch.int32) for _ in range(4))
            s["start"], s["nb"] = _zeros(17, torch.int32), _zeros(1, torch.int32)
            cap = 60 * n + 10_000                    # entries (about 26 n are kept): the same for every draw of the pairs
            s["ptr"], s["col"] = _zeros(n + 1, torch.int64), _zeros(cap, torch.int32)
            s["val"] = None if val is None else _zeros(cap)
        else:
            kept = torch.nonzero(_uniform(g, n) < 0.46).view(-1).to(torch.int32)
            s["pos"][: kept.numel()] = kept
            s["cnt"].fill_(kept.numel())
            s["loss"], s["T"] = _gamma2(g, n, 1.0), torch.full((1,), 1.7, device="cuda")
    return s


# ---------------------------------------------------------------------------
# one pass


def run(s):
    c, k = s["case"], s["case"]["kind"]
    if k == "step":
        api.fused_step(s["F"], s["y"], s["idx"], c["P"], s["w"], s["phi"], s["b"], s["cfg"], None, s["prob"],
                       s["keep"], s["pos"], s["ids"], s["loss"], s["cnt"], s["ws"])
        return {n: s[n] for n in ("w", "phi", "b", "prob", "keep", "pos", "ids", "loss", "cnt")}
    if k in ("epoch", "sparse"):
        api.train_epoch(s["F"], s["y"], s["perm"], c["n"], c["P"], s["w"], s["phi"], s["b"], s["cfg"], s["t"],
                        s["hist"], s["ws"], s["ids"], s["loss"])
        return {n: s[n] for n in ("w", "phi", "b", "t", "hist", "ids", "loss")}
    if k == "staged":
        P, ws = c["P"], s["ws"]
        api.assistant_score(s["F"], s["idx"], P, s["phi"], s["b"], None, s["prob"])
        api.shrink(s["prob"], P, GAMMA, PHILOX, 0, s["keep"], s["pos"], s["cnt"], ws)
        api.gather(s["x"], 4 * c["d"], s["idx"], s["pos"], s["cnt"], P, s["xk"], s["ids"])
        api.gather(s["y"], 4, s["idx"], s["pos"], s["cnt"], P, s["yk"], None)
        api.svm_sgd_step(s["Fk"], s["yk"], None, s["cnt"], P, s["w"], LAM, 8.0, 0.0, s["loss"], ws)
        api.assistant_update(s["Fk"], None, s["cnt"], P, s["loss"], s["T"], s["phi"], s["b"], LR_A, 0.0, ws)
        return {n: s[n] for n in ("w", "phi", "b", "prob", "keep", "pos", "ids", "loss", "cnt", "xk", "yk")}
    if k == "sk":
        api.sk_epoch(s["F"], s["y"], s["perm"], c["n"], c["P"], s["w"], s["T"], LAM, 32.0, s["t"], s["hist"],
                     s["ws"], s["ids"], s["loss"])
        return {n: s[n] for n in ("w", "t", "hist", "ids", "loss")}
    if k == "stale":
        api.train_epoch_stale(s["F"], s["y"], s["perm"], c["n"], c["P"], c["staleness"], s["w"], s["phi"], s["b"],
                              s["cfg"], s["t"], s["hist"], s["ids"], s["ws"], s["side"])
        return {n: s[n] for n in ("w", "phi", "b", "t", "hist", "ids")}
    if k == "images":
        P, B = c["P"], c["B"]
        api.score_shrink(s["F"], s["idx"], P, s["phi"], s["b"], GAMMA, 11, 0, None, s["prob"], s["keep"], s["pos"],
                         s["cnt"], s["ws"])
        api.gather(s["store"], c["row_bytes"], s["idx"], s["pos"], s["cnt"], P, s["batches"], s["ids"])
        m = int(s["cnt"].item())                     # the program has to know how many batches there are
        for lo in range(0, m, B):
            size = s["full"] if lo + B <= m else s["rest"].fill_(m - lo)
            api.threshold_assistant_update(s["F"], s["ids"][lo:], size, B, s["losses"][lo:], 0.9, s["T"], s["init"],
                                           s["phi"], s["b"], 0.05, 0.0, s["ws"])
        return {n: s[n] for n in ("phi", "b", "T", "prob", "keep", "pos", "ids", "cnt", "batches")}
    n = c["n"]
    if k == "batches":
        api.score_shrink(s["F"], None, n, s["phi"], s["b"], GAMMA, 21, 0, None, s["prob"], s["keep"], s["pos"],
                         s["cnt"], s["ws"])
        api.gather(s["ls"], 4, None, s["pos"], s["cnt"], n, s["ls_k"], None)
        api.gather(s["lt"], 4, None, s["pos"], s["cnt"], n, s["lt_k"], None)
        api.bucket_batches(s["ls_k"], s["lt_k"], s["cnt"], n, 8, 16, 4096, s["order"], s["start"], s["batch_of"],
                           s["nb"], s["ws"])
        api.gather_csr(s["F"], None, s["pos"], s["cnt"], n, s["ptr"], s["col"], s["val"], s["col"].numel(), s["ws"])
        return {name: s[name] for name in ("prob", "keep", "pos", "cnt", "ls_k", "lt_k", "order", "start", "batch_of",
                                           "nb", "ptr", "col", "val")}
    api.assistant_update(s["F"], s["pos"], s["cnt"], n, s["loss"], s["T"], s["phi"], s["b"], 0.5, 0.0, s["ws"])
    return {"phi": s["phi"], "b": s["b"]}


# ---------------------------------------------------------------------------
# what a pass cannot do without


def work(case):
    """Rows read once, per-candidate inputs and outputs, model vectors read and written per step.
    Kept rows count with the share the inputs lead to (about 0.65 dense, 0.6 sparse, 0.55 images,
    0.46 sentence pairs)."""
    k = case["kind"]
    if k in ("step", "epoch", "sk", "stale", "staged"):
        d, P = case["d"], case["P"]
        cand = P if k in ("step", "staged") else case["n"]
        steps = 1 if k in ("step", "staged") else -(-case["n"] // P)
        vecs = 1 if k == "sk" else 2
        per = 4 * d + 4 + 4 + 0.65 * 8 + (9 if k in ("step", "staged") else 0)  # row, id, label, kept id + loss
        if k in ("stale", "staged"):
            per += 0.65 * 4 * d                     # the Boss reads the kept rows again (another model, later)
        if k == "staged":
            per += 0.65 * 4 * d                     # and gets them as a matrix of their own
        flops = cand * d * 2 * (1 + 0.65 * (3 if vecs == 2 else 1))
        return {"bytes": cand * per + steps * vecs * 8 * d, "flops": flops}
    if k == "sparse":
        n, d, z = case["n"], case["d"], case["nnz"]
        steps = -(-n // case["P"])
        return {"bytes": n * (8 * z + 16 + 8 + 0.6 * 8) + steps * 16 * d, "flops": n * z * 2 * (1 + 0.6 * 3)}
    if k == "images":
        P, d, m = case["P"], case["d"], 0.55 * case["P"]
        return {"bytes": P * (4 * d + 13) + m * (2 * case["row_bytes"] + 8) + m * (4 * d + 8) + m / case["B"] * 8 * d,
                "flops": P * d * 2 + m * d * 4}
    entry = 4 if case["ones"] else 8
    z, n, m = 54 + (0 if case["ones"] else 2), case["n"], 0.46 * case["n"]
    if k == "batches":
        return {"bytes": n * (z * entry + 8 + 5) + m * 4 + m * 16 + m * (8 + 8) + m * (2 * z * entry + 16),
                "flops": n * z * 2}
    return {"bytes": m * (z * entry + 16 + 4 + 4) + 16 * case["vocab"], "flops": m * z * 4}


def tolerance(case):
    # fp32 data, sums in fp32 or better: one step is within 2e-7 of its value in 64 bits, a chain of forty
    # within 2e-7 too, but there a rounding may put a loss on the other side of its threshold.  Whole
    # numbers are the same (a draw within rounding of its probability is rare at these sizes).
    chained = case["kind"] in ("epoch", "sparse", "sk", "stale", "images")
    return {"rel": 1e-5, "max": 1e-3} if chained else {"rel": 2e-6, "max": 1e-4}


# ---------------------------------------------------------------------------
# the same pass in 64 bits


def _draws(P, seed, step):
    """Philox4x32-10, counter (j, 0, step), key seed: first word as a uniform on the 2^-24 grid."""
    m32 = 0xFFFFFFFF
    j = torch.arange(P, dtype=torch.int64, device="cuda")
    c = [j, torch.zeros_like(j), torch.full_like(j, step & m32), torch.full_like(j, step >> 32)]
    k0, k1 = seed & m32, seed >> 32
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57   # modulo 2^64: all 64 bits of the product are there
        c = [((p1 >> 32) & m32) ^ c[1] ^ k0, p1 & m32, ((p0 >> 32) & m32) ^ c[3] ^ k1, p0 & m32]
        k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
    return (c[0] >> 8).double() * 2.0 ** -24


def _kept(prob, seed, step):
    gamma = torch.tensor([GAMMA], dtype=torch.float32, device="cuda")
    return _draws(prob.numel(), seed, step) < gamma.double() + (1.0 - gamma).double() * prob


class _Rows:
    """Products with rows of the features, in 64 bits."""

    def __init__(self, s):
        self.x, self.rows, self.d = s.get("x"), s.get("rows"), s["F"].d

    def take(self, ids):
        ids = ids.long()
        if self.x is not None:
            return self.x[ids, : self.d].double()
        ptr, col, val = self.rows
        lo, have = ptr[ids], ptr[ids + 1] - ptr[ids]
        first = torch.cumsum(have, 0) - have
        row = torch.repeat_interleave(torch.arange(ids.numel(), device="cuda"), have)
        at = lo[row] + torch.arange(row.numel(), device="cuda") - first[row]
        return ids.numel(), row, col[at].long(), None if val is None else val[at].double()

    def dot(self, t, v):
        if self.x is not None:
            return t @ v
        n, row, col, val = t
        return torch.zeros(n, dtype=torch.float64, device="cuda").index_add_(0, row, v[col] if val is None else val * v[col])

    def add(self, t, coef):
        """Sum of the rows, each times its coefficient."""
        if self.x is not None:
            return coef @ t
        n, row, col, val = t
        out = torch.zeros(self.d, dtype=torch.float64, device="cuda")
        return out.index_add_(0, col, coef[row] if val is None else val * coef[row])


class _Model:
    def __init__(self, s):
        self.w, self.phi, self.b = (s[n].double().clone() if n in s else None for n in ("w", "phi", "b"))
        self.T, self.t = s["T"].double(), 0

    def boss(self, R, t, y, lr):
        """SVM step on the rows of t; their losses at the old w."""
        margin = y * R.dot(t, self.w)
        coef = torch.where(margin < 1, y, 0.0)
        self.w = (1 - lr * LAM) * self.w + lr / y.numel() * R.add(t, coef)
        return (1 - margin).clamp(min=0)

    def assistant(self, R, t, loss, lr_a, T=None):
        z = (loss > (self.T if T is None else T)).double()
        resid = torch.sigmoid(R.dot(t, self.phi) + self.b) - z
        self.phi = self.phi - lr_a / resid.numel() * R.add(t, resid)
        self.b = self.b - lr_a * resid.mean()

    def lr(self, lr0):
        self.t += 1
        return lr0 / math.sqrt(self.t)


def _front(size, values):
    out = torch.zeros(size, dtype=torch.float64, device="cuda")
    out[: values.numel()] = values
    return out


def exact(case, seed):
    s, k = prepare(case, seed), case["kind"]
    if k in ("step", "staged"):
        P, R, M = case["P"], _Rows(s), _Model(s)
        prob = torch.cat([torch.sigmoid(R.dot(R.take(i), M.phi) + M.b) for i in s["idx"].split(65_536)])
        ids = s["idx"][_kept(prob, PHILOX, 0)]
        t, y = R.take(ids), s["y"][ids.long()].double()
        phi = M.phi
        loss = M.boss(R, t, y, 8.0)
        M.phi = phi
        M.assistant(R, t, loss, LR_A)
        out = {n: None for n in ("keep", "pos", "ids", "cnt")}
        out.update(w=M.w, phi=M.phi, b=M.b, prob=prob, loss=_front(P, loss))
        if k == "staged":
            out["xk"], out["yk"] = _front(P * case["d"], t.reshape(-1)).view(P, -1), _front(P, y)
        return out
    if k in ("epoch", "sparse", "sk", "stale"):
        n, P, R, M = case["n"], case["P"], _Rows(s), _Model(s)
        lr0, losses, old = 4.0 if k == "sparse" else 32.0, [], []
        for step, idx in enumerate(s["perm"].split(P)):
            t, y = R.take(idx), s["y"][idx.long()].double()
            if k == "sk":
                keep = (1 - y * R.dot(t, M.w)).clamp(min=0) > M.T
            else:
                old.append((M.phi, M.b))             # the Assistant after `step` updates
                phi, b = old[max(0, step - case.get("staleness", 0))]
                keep = _kept(torch.sigmoid(R.dot(t, phi) + b), PHILOX, step)
            ids = idx[keep]
            if ids.numel() == 0:
                losses.append(_front(P, ids.double()))
                continue
            t, y = R.take(ids), y[keep]
            loss = M.boss(R, t, y, M.lr(lr0))
            if k != "sk":
                M.assistant(R, t, loss, LR_A)
            losses.append(_front(P, loss))
        out = {"w": M.w, "t": None, "hist": None, "ids": None}
        if k != "sk":
            out.update(phi=M.phi, b=M.b)
        if k != "stale":
            out["loss"] = torch.cat(losses)
        return out
    if k == "images":
        R, M, B = _Rows(s), _Model(s), case["B"]
        prob = torch.sigmoid(R.dot(R.take(s["idx"]), M.phi) + M.b)
        ids = s["idx"][_kept(prob, 11, 0)]
        T = None
        for lo in range(0, ids.numel(), B):
            part = ids[lo:lo + B]
            loss = s["losses"][lo:lo + part.numel()].double()
            mid = loss.sort()[0]
            med = (mid[(mid.numel() - 1) // 2] + mid[mid.numel() // 2]) / 2
            T = med if T is None else 0.9 * T + 0.1 * med
            M.assistant(R, R.take(part), loss, 0.05, T)
        out = {n: None for n in ("keep", "pos", "ids", "cnt", "batches")}
        out.update(phi=M.phi, b=M.b, T=T.view(1), prob=prob)
        return out
    R = _Rows(s)
    if k == "batches":
        out = {n: None for n in ("keep", "pos", "cnt", "ls_k", "lt_k", "order", "start", "batch_of", "nb", "ptr", "col",
                                 "val")}
        every = torch.arange(case["n"], device="cuda")
        out["prob"] = torch.cat([torch.sigmoid(R.dot(R.take(i), s["phi"].double()) + s["b"].double())
                                 for i in every.split(131_072)])
        return out
    M, m = _Model(s), int(s["cnt"].item())
    M.assistant(R, R.take(s["pos"][:m]), s["loss"][:m].double(), 0.5)
    return {"phi": M.phi, "b": M.b}
