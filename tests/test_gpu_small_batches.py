"""GPU parity of the passes over small batches of chosen rows (at most 512: a lane group for each row)."""
import pytest
import torch

from paper_1905_03381_amd import api

import test_gpu_dense as dense
from gpu_util import scalar_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ws():
    return api.Workspace(4000, 2048)


# every lane layout, at batch sizes around the number of rows of a wave, a block and the whole range
# (the Boss step gets room for five rows more than there are)
@pytest.mark.parametrize("n,d,ld,m", [(600, 64, None, 1), (600, 36, None, 507), (600, 128, None, 257), (600, 200, 256, 256),
                                      (600, 512, None, 255), (600, 1000, None, 506), (600, 1024, None, 507),
                                      (600, 2048, None, 64), (600, 2048, None, 508)])
def test_small_batches_match_the_oracle(ref, ws, n, d, ld, m):
    dense.test_svm_sgd_step(ref, ws, n, d, ld, m, False)
    dense.test_assistant_update(ref, ws, n, d, ld, m)


@pytest.mark.parametrize("m", [3, 256, 257, 512])
def test_batch_median_beside_infinite_losses_and_rows(m):
    """Infinite losses have a rank; a row past the batch (infinite here) is read by no sum."""
    d = 128
    g = torch.Generator().manual_seed(m)
    x, loss = torch.randn(600, d, generator=g).cuda(), torch.rand(m, generator=g).cuda()
    x[m:] = float("inf")
    loss[0] = float("inf")
    F, cnt = api.Features.dense(x), scalar_dev(m, torch.int32)
    one, two = ((torch.full((d,), 0.1, device="cuda"), scalar_dev(0.0), scalar_dev(0.0), scalar_dev(0, torch.int32))
                for _ in "ab")
    ws = api.Workspace(512, d)
    api.threshold_assistant_update(F, None, cnt, 512, torch.cat([loss, loss[:512 - m]]) if m < 512 else loss, 0.9, one[2],
                                   one[3], one[0], one[1], 0.5, 0.0, ws)
    api.threshold_update(loss, cnt, m, 0.9, two[2], two[3])
    api.assistant_update(F, None, cnt, m, loss, two[2], two[0], two[1], 0.5, 0.0, ws)
    mid = loss.sort()[0]
    med = mid[m // 2] if m % 2 else (mid[m // 2 - 1] + mid[m // 2]) * 0.5
    assert torch.equal(one[2], med.view(1)) and torch.equal(two[2], one[2])
    assert torch.isfinite(one[0]).all()
    # (a different room for the batch spreads it over other blocks: fp32 sums of m terms of size 1/m)
    assert torch.allclose(one[0], two[0], rtol=0, atol=1e-6) and torch.allclose(one[1], two[1], rtol=0, atol=1e-6)


@pytest.mark.parametrize("d", [36, 100, 128, 200, 260, 1000, 1028])
@pytest.mark.parametrize("m", [1, 9, 300])
def test_infinite_model_entries_at_the_end_of_the_row(d, m):
    """An infinite entry of w in the last columns gives infinite losses with the signs of the features: lanes
    past the end of a row, which hold its last piece again, add nothing."""
    X = torch.randn(m, d, generator=torch.Generator().manual_seed(d)).cuda()
    w = torch.full((d,), 0.01, device="cuda")
    w[d - 2] = float("inf")
    sign, loss = torch.sign(X[:, d - 2]), torch.zeros(m, device="cuda")
    api.svm_sgd_step(api.Features.dense(X), torch.ones(m, device="cuda"), None, torch.full((1,), m, dtype=torch.int32, device="cuda"),
                     m, w, 0.0, 0.0, 0.0, loss, api.Workspace(m, d))
    assert torch.equal(loss, torch.where(sign > 0, 0.0, float("inf")))
