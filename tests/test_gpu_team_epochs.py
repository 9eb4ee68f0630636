"""GPU parity of epochs over small pools that a team of blocks runs: every step against the oracle's step from the GPU's
previous state, then the epoch in one call, bit for bit (single steps are done by one block)."""
import numpy as np
import pytest
import torch

from paper_1905_03381_amd import api

from gpu_util import dense_features, dev, host, scalar_dev
from stepwise import check_epoch

pytestmark = pytest.mark.gpu

# third control word of a workspace (csrc/aa_small.hpp): SHUT: its epochs are done by one block; 4 (t + 1) + b: block b
# leaves in step t.  The gate's states have the same numbers.
OPEN, SHUT = 1, 2


def _problem(n, d, ld=None):
    r = np.random.default_rng(d)
    X = r.standard_normal((n, ld or d)).astype(np.float32)
    X /= np.linalg.norm(X[:, :d], axis=1, keepdims=True)
    y = np.where(X[:, :d] @ r.standard_normal(d) > 0, 1.0, -1.0).astype(np.float32)
    return X, y, r.permutation(n).astype(np.int32), (0.8 * r.standard_normal(d)).astype(np.float32)


def _workspace(P, d, alone, ends=None):
    ws = api.Workspace(P, d)
    if alone or ends is not None:
        off = ws.ptr - ws.buf.data_ptr()
        ws.buf[off:off + 256].view(torch.int32)[2] = SHUT if ends is None else ends
    return ws


def _gate(ws):
    """Blocks that were there, state of the gate, blocks that got through, of the last epoch that had a team."""
    return host(_gate_words(ws)).tolist()


def _gate_words(ws):
    first = ws.ptr - ws.buf.data_ptr() + 256 + 2 * 4 * 1024 + 256  # (the gradients' part of the workspace)
    return ws.buf[first:first + 12].view(torch.int32)


def _has_team(d, P, n, hard):
    """The rule of launch_team (csrc/aa_small.hip): more than two turns of rows a wave, or soft keeps and rows narrower than a
    wave, and 32 turns in all."""
    lanes = 16 if d <= 64 else 32 if d <= 128 else 64
    rows = 16 * (64 // lanes)
    turns = 2 if P <= 2 * rows else 4 if P <= 4 * rows else 8
    return (turns > 2 or (not hard and lanes < 64)) and -(-n // P) * turns >= 32


# every lane layout at its first and last width and every number of turns, waves without rows, the smallest number of steps
# of a team, odd and even, last pools of one row
@pytest.mark.parametrize("d,P,n,ld", [(4, 17, 273, None), (64, 128, 2048, 68), (64, 129, 1033, None), (60, 512, 1537, None),
                                      (68, 50, 801, None), (128, 65, 521, 132), (128, 256, 1100, None), (132, 33, 265, None),
                                      (256, 64, 512, None), (200, 65, 196, None), (256, 128, 640, None)])
@pytest.mark.parametrize("hard", [False, True])
@pytest.mark.parametrize("alone", [False, True])
def test_teams(ref, d, P, n, ld, hard, alone):
    X, y, perm, w0 = _problem(n, d, ld)
    ws = _workspace(P, d, alone)
    _gate_words(ws).fill_(-7)
    counts, _ = check_epoch(ref, ref.Features.dense(X, d=d), dense_features(X, d=d), y, perm, n, P, w0,
                            None if hard else w0[::-1].copy(), 0.1, gamma=0.0 if hard else 0.2, seed=5, step0=3, lam=1e-3,
                            lr0=0.5, lr_a=0.3, T=0.4, ws=ws, hard=hard)
    assert len(counts) == -(-n // P)
    # (the steps one a call have no team, the epoch has: the same bits do not tell who made them)
    assert _gate(ws) == ([-7] * 3 if not _has_team(d, P, n, hard) else [4, SHUT, 0] if alone else [4, OPEN, 4])


# early, late, and in the last step, when the other blocks have all they need: block 0, which tells the counts, and another
@pytest.mark.parametrize("step,block", [(0, 1), (4, 0), (5, 3), (19, 0), (19, 2)])
@pytest.mark.parametrize("d,P,hard", [(128, 256, False), (200, 128, False), (64, 300, True)])
def test_team_that_loses_a_block(d, P, hard, step, block):
    """A block whose wait for words has passed its limit leaves: the epoch is then done by one block, with the same bits
    everywhere, and nothing of the team's is left in the model."""
    n = 20 * P - 7
    X, y, perm, w0 = _problem(n, d)
    F, yd, pd, T = dense_features(X), dev(y), dev(perm), scalar_dev(0.4)
    got = []
    for ws in (_workspace(P, d, True), _workspace(P, d, False, ends=4 * (step + 1) + block)):
        w, phi, b, tu = dev(w0), dev(w0), scalar_dev(0.1), torch.full((1,), 3, dtype=torch.int32, device="cuda")
        hist = torch.full((20,), -1, dtype=torch.int32, device="cuda")
        ids, loss = torch.full((20, P), -1, dtype=torch.int32, device="cuda"), torch.full((20, P), -3.0, device="cuda")
        if hard:
            api.sk_epoch(F, yd, pd, n, P, w, T, 1e-3, 0.5, tu, hist, ws, ids, loss)
        else:
            cfg = api.step_config(0.2, 1e-3, 0.5, 0.3, 0.01, 5, 0, T)
            api.train_epoch(F, yd, pd, n, P, w, phi, b, cfg, tu, hist, ws, ids, loss)
        got.append([host(t).copy() for t in (w, phi, b, tu, hist, ids, loss)])
        there, state, through = _gate(ws)
    assert there == 4 and state == OPEN and through == (3 if step == 19 else 0)
    assert all(np.array_equal(u, v) for u, v in zip(*got))
    assert (got[0][4] > 0).all() and got[0][3][0] == 23 and not np.array_equal(got[0][0], w0)


def test_workspace_without_room_for_the_words():
    """A workspace as small as one block needs is still taken, with the same results."""
    d, P, n = 64, 16, 400
    X, y, perm, w0 = _problem(n, d)
    F, yd, pd, T = dense_features(X), dev(y), dev(perm), scalar_dev(0.4)
    got = []
    for small in (False, True):
        ws = _workspace(P, d, False)
        if small:
            ws.bytes = 30_000
        w, phi, b = dev(w0), dev(w0), scalar_dev(0.1)
        _gate_words(ws).fill_(-7)
        api.train_epoch(F, yd, pd, n, P, w, phi, b, api.step_config(0.2, 1e-3, 0.5, 0.3, 0.01, 5, 0, T), None, None, ws)
        assert _gate(ws) == ([-7] * 3 if small else [4, OPEN, 4])
        got.append((host(w), host(phi), host(b)))
    assert all(np.array_equal(u, v) for u, v in zip(*got)) and not np.array_equal(got[0][0], w0)


@pytest.mark.parametrize("alone", [False, True])
def test_graph_replays(alone):
    """Without histories, bias and step-size counter; captured and replayed with other work in between."""
    d, P, n = 128, 256, 5000
    X, y, perm, w0 = _problem(n, d)
    F, yd, pd, ws, T = dense_features(X), dev(y), dev(perm), _workspace(P, d, alone), scalar_dev(0.4)
    cfg = api.step_config(0.2, 1e-3, 0.5, 0.3, 0.01, 5, 0, T)
    w, phi = dev(w0), dev(w0)
    want = []
    for _ in range(4):
        api.train_epoch(F, yd, pd, n, P, w, phi, None, cfg, None, None, ws)
        want.append((host(w).copy(), host(phi).copy()))
    assert np.isfinite(want[3][0]).all() and not np.array_equal(want[0][0], w0)
    w, phi = dev(w0), dev(w0)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            api.train_epoch(F, yd, pd, n, P, w, phi, None, cfg, None, None, ws)
    for k in range(4):
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(host(w), want[k][0]) and np.array_equal(host(phi), want[k][1])
        assert _gate(ws) == ([4, SHUT, 0] if alone else [4, OPEN, 4])
        dev(w0).mul_(2)


def test_streams():
    """Epochs on several streams at once: the results of one alone."""
    d, P, n = 128, 256, 5000
    X, y, perm, w0 = _problem(n, d)
    F, yd, pd, T = dense_features(X), dev(y), dev(perm), scalar_dev(0.4)
    cfg = api.step_config(0.2, 1e-3, 0.5, 0.3, 0.01, 5, 0, T)
    streams = [torch.cuda.Stream() for _ in range(4)]
    sets = [(dev(w0), dev(w0), _workspace(P, d, False)) for _ in range(5)]
    torch.cuda.synchronize()
    for _ in range(5):
        api.train_epoch(F, yd, pd, n, P, sets[4][0], sets[4][1], None, cfg, None, None, sets[4][2])
    torch.cuda.synchronize()
    for _ in range(5):
        for s, (w, phi, ws) in zip(streams, sets):
            with torch.cuda.stream(s):
                api.train_epoch(F, yd, pd, n, P, w, phi, None, cfg, None, None, ws)
    torch.cuda.synchronize()
    assert _gate(sets[4][2]) == [4, OPEN, 4]
    for w, phi, ws in sets[:4]:
        assert _gate(ws) in ([4, OPEN, 4], [4, SHUT, 0])  # (the blocks of four teams may not all be there at once)
        assert np.array_equal(host(w), host(sets[4][0])) and np.array_equal(host(phi), host(sets[4][1]))
