"""The order-statistic projection of tensors that one workgroup or a few tiles hold, bit for bit against the oracle: element counts around
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


def _step(n, seed):
    rng = np.random.Generator(np.random.Philox(seed))
    d = (rng.standard_normal(n) * np.exp(rng.standard_normal(n)) * 1e-6).astype(np.float32)
    d[rng.integers(0, n, n // 16)] = d[rng.integers(0, n, n // 16)]          # ties
    a = np.sort(np.abs(d))
    P = [1] + list(range(5, 100, 5)) + [99, 100]
    base = np.array([a[min(n - 1, int(n * p / 100))] for p in P])
    return d, {name: (base * f).astype(np.float32) for name, f in
               (("none", 100.0), ("few", np.where(np.arange(22) < 18, 10, 0.5)), ("half", np.where(np.arange(22) % 4 < 2, 1.5, 0.7)), ("all", 0.5))}


# tiles (4096 elements) whose counters a scatter pass adds up itself, up to 64, and one more
@pytest.mark.parametrize("n", [MOST + 1, 5 * 4096, 33 * 4096 + 1, 64 * 4096, 64 * 4096 + 1])
def test_empirical_of_few_tiles(tao, oracle_mod, n):
    """Scratch memory that held anything before, and replays of a captured call on other data."""
    d, tables = _step(n, n)
    x = torch.from_numpy(d).cuda()
    out = torch.empty_like(x)
    ws = torch.full((tao.tao_project_workspace_bytes(n),), 255, dtype=torch.uint8, device="cuda")
    for name, thr in tables.items():
        tao.tao_project_empirical(x, torch.from_numpy(thr).cuda(), 1.0, out=out, ws=ws)
        assert _same(out.cpu().numpy(), oracle_mod.project_empirical(d, thr, 1.0)), name
    t = torch.from_numpy(tables["few"]).cuda()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        tao.tao_project_empirical(x, t, 1.0, out=out, ws=ws)
    for seed in range(3):
        d2, tables2 = _step(n, n + 1 + seed)
        x.copy_(torch.from_numpy(d2)); t.copy_(torch.from_numpy(tables2["half" if seed % 2 else "few"]))
        ws.fill_(seed)
        g.replay()
        assert _same(out.cpu().numpy(), oracle_mod.project_empirical(d2, tables2["half" if seed % 2 else "few"], 1.0)), seed


@pytest.mark.parametrize("n", [1, 4096, 4097, 300001, 1048577])
def test_profile_of_errors_with_used_scratch(tao, n):
    """The last workgroup of the reduction has the ratios: the same bytes whatever the scratch memory held, call after call and replayed."""
    import ctypes
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    c, r = torch.randn(n, generator=g, device="cuda"), torch.randn(n, generator=g, device="cuda")
    thr = torch.rand(22, generator=g, device="cuda") * 0.2 + 0.9
    ws = torch.zeros(tao.tao_profile_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    out = torch.zeros(ctypes.sizeof(tao.ErrorProfile), dtype=torch.uint8, device="cuda")
    first = tao.tao_profile_errors(c, r, thr_abs=thr, thr_rel=thr, out=out, ws=ws).copy()
    d = (c.double() - r.double()).abs()
    assert first["max_abs"] == d.float().max().item() and first["n"] == n
    ratios = [float(first[k][i]) / float(thr[i].item()) for k in ("abs_p", "rel_p") for i in range(22)]
    assert first["p_max"] == max(ratios)
    want = out.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        tao.tao_profile_errors(c, r, thr_abs=thr, thr_rel=thr, out=out, ws=ws, readback=False)
    for fill in (255, 1, 0, 63):
        ws.fill_(fill); out.fill_(fill)
        tao.tao_profile_errors(c, r, thr_abs=thr, thr_rel=thr, out=out, ws=ws, readback=False)
        assert torch.equal(out, want)
        ws.fill_(fill); out.fill_(fill)
        graph.replay()
        assert torch.equal(out, want)
