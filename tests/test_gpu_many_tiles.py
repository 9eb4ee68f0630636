"""Compaction, CSR assembly and length buckets on both sides of the numbers of tiles up to which every block
adds up the counts before its own, and CSR rows around the four entries a lane copies at a time.  All
outputs are whole numbers or copies: compared exactly, with torch on the device."""
import pytest
import torch

from paper_1905_03381_amd import api

from gpu_util import scalar_dev

pytestmark = pytest.mark.gpu


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _zeros(n, dtype=torch.int32):
    return torch.zeros(n, dtype=dtype, device="cuda")


@pytest.mark.parametrize("P", [(1 << 18) + 1, 300 * 2048 + 5, 4096 * 2048, 4096 * 2048 + 1, 8192 * 2048,
                               8192 * 2048 + 1])
def test_shrink_threshold_over_many_tiles(P):
    crit = torch.rand(P, generator=_gen(P), device="cuda")
    keep, pos, cnt = _zeros(P, torch.uint8), _zeros(P), _zeros(1)
    api.shrink_threshold(crit, P, scalar_dev(0.7), keep, pos, cnt, api.Workspace(P, 4))
    want = torch.nonzero(crit > torch.tensor(0.7, device="cuda")).view(-1).to(torch.int32)
    assert torch.equal(keep.bool(), crit > 0.7) and int(cnt) == want.numel()
    assert torch.equal(pos[:want.numel()], want) and not pos[want.numel():].any()


@pytest.mark.parametrize("n,most", [(1025, 9), (5000, 140), (200_000, 70), (2048 * 1024, 5), (2048 * 1024 + 1, 5),
                                    (8192 * 1024, 3), (8192 * 1024 + 1025, 5)])
@pytest.mark.parametrize("ones", [False, True])
def test_csr_assembly(n, most, ones):
    g = _gen(n)
    length = torch.randint(0, most + 1, (n,), generator=g, device="cuda")
    ptr = _zeros(n + 1, torch.int64)
    ptr[1:] = torch.cumsum(length, 0)
    nnz = int(ptr[-1])
    col = torch.randint(0, 1 << 30, (nnz,), generator=g, device="cuda", dtype=torch.int32)
    val = None if ones else torch.rand(nnz, generator=g, device="cuda")
    kept = torch.nonzero(torch.rand(n, generator=g, device="cuda") < 0.9).view(-1)
    idx = torch.randperm(n, generator=g, device="cuda")
    m, rows = kept.numel(), idx[kept]
    have = length[rows]
    want_ptr = _zeros(m + 1, torch.int64)
    want_ptr[1:] = torch.cumsum(have, 0)
    total = int(want_ptr[-1])
    at = torch.repeat_interleave(ptr[rows] - want_ptr[:-1], have) + torch.arange(total, device="cuda")
    out_ptr, out_col = torch.full((n + 1,), -1, dtype=torch.int64, device="cuda"), _zeros(nnz + 1)
    out_val = None if ones else _zeros(nnz + 1, torch.float32)
    F, pos, cnt, ws = api.Features.csr(ptr, col, val, 1 << 30), kept.to(torch.int32), scalar_dev(m, torch.int32), None
    ws = api.Workspace(n, 4)
    api.gather_csr(F, idx.to(torch.int32), pos, cnt, n, out_ptr, out_col, out_val, nnz + 1, ws)
    assert torch.equal(out_ptr[:m + 1], want_ptr) and bool((out_ptr[m + 1:] == -1).all())
    assert torch.equal(out_col[:total], col[at]) and not out_col[total:].any()
    if not ones:
        assert torch.equal(out_val[:total], val[at]) and not out_val[total:].any()
    # rows that do not fit are not copied, the pointers stay whole
    cap = total // 2
    out_col.zero_()
    api.gather_csr(F, idx.to(torch.int32), pos, cnt, n, out_ptr, out_col, out_val, cap, ws)
    fit = int((want_ptr <= cap).sum()) - 1
    end = int(want_ptr[fit])
    assert torch.equal(out_ptr[:m + 1], want_ptr)
    assert torch.equal(out_col[:end], col[at][:end]) and not out_col[end:].any()


@pytest.mark.parametrize("m_max", [2047, 1024 * 2048, 1024 * 2048 + 1])
@pytest.mark.parametrize("n_buckets", [1, 16, 32])
def test_buckets_over_many_tiles(m_max, n_buckets):
    g = _gen(m_max + n_buckets)
    ls, lt = (torch.randint(1, 130, (m_max,), generator=g, device="cuda", dtype=torch.int32) for _ in "st")
    m, width, budget = m_max - 3, 4, 1000
    order, batch_of, start, nb = _zeros(m_max), _zeros(m_max), _zeros(n_buckets + 1), _zeros(1)
    api.bucket_batches(ls, lt, scalar_dev(m, torch.int32), m_max, width, n_buckets, budget, order, start, batch_of, nb,
                       api.Workspace(m_max, 4))
    bucket = ((torch.maximum(ls, lt)[:m] - 1) // width).clamp(max=n_buckets - 1)
    want = torch.sort(bucket, stable=True)
    sizes = torch.bincount(bucket, minlength=n_buckets)
    first = torch.cumsum(sizes, 0) - sizes
    cap = torch.tensor([max(1, budget // (2 * width * (b + 1))) for b in range(n_buckets)], device="cuda")
    batches = (sizes + cap - 1) // cap
    base = torch.cumsum(batches, 0) - batches
    b = want.values.long()
    assert torch.equal(order[:m], want.indices.to(torch.int32))
    assert start.tolist() == first.tolist() + [m] and int(nb) == int(batches.sum())
    assert torch.equal(batch_of[:m].long(), base[b] + (torch.arange(m, device="cuda") - first[b]) // cap[b])
