"""The order-statistic projection of tensors that one workgroup holds, bit for bit against the oracle: element counts around
what a wavefront, a thread's items and the whole workgroup hold, and candidate counts around the same edges."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

MOST = 16384                                                # held by one workgroup of 1024 threads


@pytest.fixture(scope="module")
def tao():
    import paper_2510_16028_amd as t
    t.lib()
    assert torch.cuda.is_available()
    return t


def _same(got, want):
    nan = np.isnan(want)
    return np.array_equal(np.isnan(got), nan) and np.array_equal(got.view(np.uint32)[~nan], want.view(np.uint32)[~nan])


@pytest.mark.parametrize("n", [1, 3, 64, 1023, 1024, 1025, 4097, 8192, 15361, MOST - 1, MOST, MOST + 1])
@pytest.mark.parametrize("candidates", [0, 1, 65, 1024, 1025, 7000, MOST])
def test_empirical_in_one_workgroup(tao, oracle_mod, n, candidates):
    """Small magnitudes below wide thresholds, `candidates` large ones (ties, both signs, the highest index with its sign) above theirs."""
    count = min(candidates, n)
    rng = np.random.Generator(np.random.Philox(n + candidates))
    d = (rng.standard_normal(n) * 1e-6).astype(np.float32)
    at = rng.permutation(n)[:count]
    if count:
        at[0] = n - 1
        d[at] = np.where(rng.random(count) < 0.3, 1.25, 1 + rng.random(count)) * np.where(rng.random(count) < 0.5, -1, 1)
        d[n - 1] = -d[n - 1]
    if n > 64:
        d[:4] = [np.inf, -np.inf, np.nan, -0.0]
    share = 1 - count / n
    thr = np.array([1e-3 if p / 100 < share else 0.5 + p / 200 for p in [1] + list(range(5, 100, 5)) + [99, 100]], np.float32)
    want = oracle_mod.project_empirical(d, thr, 1.0)
    x = torch.from_numpy(d).cuda()
    t = torch.from_numpy(thr).cuda()
    assert _same(tao.tao_project_empirical(x, t, 1.0).cpu().numpy(), want)
    shifted = torch.zeros(n + 1, device="cuda")[1:].copy_(x)            # 4-byte aligned, in place
    assert _same(tao.tao_project_empirical(shifted, t, 1.0, out=shifted).cpu().numpy(), want)
