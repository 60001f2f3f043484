"""Quick settlement of the check (binary32 estimates, exact arithmetic only where they do not decide): the profile of the
one-pass softmax check against bound and streaming check on the CPU's own arithmetic, field for field, with errors on bin
edges, bounds just met and just missed, masked halves, and values no estimate can settle."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tao():
    import paper_2510_16028_amd as t
    t.lib()
    assert torch.cuda.is_available()
    return t


def _claims(y, tau, g):
    """Claims around y: equal, off by powers of two of y and of the bound (errors on and next to bin edges), at the bound."""
    yd, td = y.double(), tau.double()
    pick = torch.randint(0, 8, y.shape, generator=g, device=y.device)
    k = torch.randint(-30, -16, y.shape, generator=g, device=y.device).double()
    edge = yd * (1 + torch.exp2(k) * (1 + torch.randint(0, 8, y.shape, generator=g, device=y.device) / 8))
    noise = yd + td * (2 * torch.rand(y.shape, generator=g, device=y.device, dtype=torch.float64) - 1) * 0.9
    c = torch.where(pick < 3, noise, torch.where(pick < 5, edge, torch.where(pick == 5, yd + td, torch.where(pick == 6, yd + 1.000001 * td, yd))))
    return c.float()


# both sides of the rules on rows (four per row group), row lengths (wavefront, wide group) and whole vectors
@pytest.mark.parametrize("rows,cols", [(16384, 128), (16383, 200), (16384, 511), (16384, 1024), (16385, 1021), (16384, 1028),
                                       (16384, 2048), (16384, 1500), (4096, 1030), (4096, 2046), (2048, 4096), (1024, 8190)])
@pytest.mark.parametrize("alpha,eps_rel", [(1.0, 1e-12), (2.0, 0.0)])
def test_profile_equals_bound_and_streaming_check(tao, rows, cols, alpha, eps_rel):
    g = torch.Generator(device="cuda").manual_seed(rows + cols)
    x = torch.randn((rows, cols), generator=g, device="cuda")
    if cols % 2 == 0:
        x.masked_fill_(torch.arange(cols, device="cuda")[None] > torch.arange(rows, device="cuda")[:, None] % cols, float("-inf"))
        x[::5] = x[::5].clamp(min=-3.0e38)                   # masks of (nearly) the lowest finite value as well
    y = torch.softmax(x, -1)
    tau = tao.tao_bound_softmax(x, y)
    c = _claims(y, tau, g)
    c[3, 5] = float("nan"); c[rows - 1, cols - 1] = float("inf"); y[7, 1] = 0.0; c[7, 1] = 1e-40; x[11, 2] = float("nan")
    tau = tao.tao_bound_softmax(x, y)
    want = tao.tao_check_and_profile(c, y, tau, alpha=alpha, eps_rel=eps_rel)
    got = tao.tao_bound_check_softmax(x, y, c, alpha=alpha, eps_rel=eps_rel)
    assert set(got) == set(want)
    for key in want:
        a, b = np.asarray(got[key]), np.asarray(want[key])
        assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f"), key


@pytest.mark.parametrize("kind", ["layernorm", "rmsnorm"])
@pytest.mark.parametrize("rows,cols", [(16384, 200), (16390, 511), (8192, 768), (8191, 1021), (8192, 1024), (8200, 1030), (4096, 4096), (2049, 8190), (300, 8200)])
def test_norm_profile_equals_bound_and_streaming_check(tao, kind, rows, cols):
    g = torch.Generator(device="cuda").manual_seed(rows + cols)
    k = tao.NORM_LAYERNORM if kind == "layernorm" else tao.NORM_RMSNORM
    x = torch.randn((rows, cols), generator=g, device="cuda")
    x[::7] *= 1e30; x[1::7] *= 1e-30; x[2::7] += 1e4         # products past the range of the estimates, a cancelling mean
    gamma = 1 + 0.1 * torch.randn(cols, generator=g, device="cuda")
    d = x.double() - (x.double().mean(-1, keepdim=True) if kind == "layernorm" else 0)
    y = (d * torch.rsqrt((d * d).mean(-1, keepdim=True) + 1e-5) * gamma).float()
    tau = tao.tao_bound_norm(k, x, y, gamma, None, eps=1e-5)
    c = _claims(y, torch.nan_to_num(tau, nan=0.0, posinf=0.0), g)
    c[3, 5] = float("nan"); c[rows - 1, cols - 1] = float("inf")
    want = tao.tao_check_and_profile(c, y, tau)
    got = tao.tao_bound_check_norm(k, x, y, c, gamma, None, eps=1e-5)
    # (claims sit exactly at the bound, and the two kernels add a row in different orders: a bound on a rounding edge may fall
    # either way; the errors themselves do not depend on it)
    assert abs(got["violations"] - want["violations"]) <= rows * cols * 1e-5
    for key in set(want) - {"violations", "accept"}:
        a, b = np.asarray(got[key]), np.asarray(want[key])
        assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f"), key


@pytest.mark.parametrize("n", [4096, 4 * 1024 * 1024 - 4, 4 * 1024 * 1024, 8 * 1024 * 1024, 9 * 1024 * 1024 + 3])
@pytest.mark.parametrize("kind", ["ACT_SILU", "ACT_GELU_ERF", "ACT_GELU_TANH", "ACT_MUL", "ACT_RELU"])
def test_act_profile_equals_bound_and_streaming_check(tao, kind, n):
    g = torch.Generator(device="cuda").manual_seed(n)
    k = getattr(tao, kind)
    x = 3 * torch.randn(n, generator=g, device="cuda")
    x[5::1001] *= 1e30; x[6::1001] *= 1e-40
    xd = x.double()
    y = (xd / (1 + torch.exp(-xd)) if kind == "ACT_SILU" else 0.5 * xd * (1 + torch.erf(xd * 0.5 ** 0.5)) if "GELU" in kind else xd).float()
    tau = tao.tao_bound_act(k, x, y, x2=x)
    c = _claims(y, torch.nan_to_num(tau, nan=0.0, posinf=0.0), g)
    c[3] = float("nan"); c[n - 1] = float("inf"); x[11] = float("nan"); x[12] = float("inf")
    tau = tao.tao_bound_act(k, x, y, x2=x)
    want = tao.tao_check_and_profile(c, y, tau)
    got = tao.tao_bound_check_act(k, x, y, c, x2=x)
    for key in want:
        a, b = np.asarray(got[key]), np.asarray(want[key])
        assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f"), key


# alphas under which the estimates must settle nothing: the softmax check takes any alpha, like the streaming check (whose
# comparison fails for NaN everywhere, and for an infinite alpha where the bound is 0)
@pytest.mark.parametrize("alpha", [float("nan"), float("inf"), -1.0, 0.0, 2.0 ** -40, 2.0 ** 40, 1e300])
@pytest.mark.parametrize("rows,cols", [(16384, 128), (16384, 1024), (16384, 2048)])
def test_alphas_that_are_no_ordinary_factor(tao, rows, cols, alpha):
    g = torch.Generator(device="cuda").manual_seed(rows + cols)
    x = torch.randn((rows, cols), generator=g, device="cuda")
    x.masked_fill_(torch.arange(cols, device="cuda")[None] > torch.arange(rows, device="cuda")[:, None] % cols, float("-inf"))
    y = torch.softmax(x, -1)
    tau = tao.tao_bound_softmax(x, y)
    c = _claims(y, tau, g)
    want = tao.tao_check_and_profile(c, y, tau, alpha=alpha)
    got = tao.tao_bound_check_softmax(x, y, c, alpha=alpha)
    for key in want:
        a, b = np.asarray(got[key]), np.asarray(want[key])
        assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f"), key


# Rows at which a binary32 estimate of the bound would be formed from subnormal numbers.  Claims lie 2^-14 ... 2^-8 of the
# bound inside and outside it (y = 0, so that they can): far beyond the last bit, in which the two kernels' bounds may differ.
@pytest.mark.parametrize("kind,rows_are", [("rmsnorm", "tiny products"), ("rmsnorm", "huge"), ("layernorm", "huge"), ("layernorm", "subnormal"),
                                           ("rmsnorm", "subnormal")])
@pytest.mark.parametrize("rows,cols", [(16384, 512), (16384, 511), (16384, 1024)])
def test_norm_rows_at_the_ends_of_the_range(tao, kind, rows_are, rows, cols):
    g = torch.Generator(device="cuda").manual_seed(rows + cols)
    k = tao.NORM_LAYERNORM if kind == "layernorm" else tao.NORM_RMSNORM
    rand = lambda: torch.rand((rows, cols), generator=g, device="cuda")
    gamma = torch.ones(cols, device="cuda")
    if rows_are == "tiny products":
        x = 1e-30 * (0.5 + rand())
        x[:, ::8] *= 1e-6; gamma[::8] = 1e-6                 # x g about 1e-42
    elif rows_are == "huge":
        x = 3e38 * (2 * rand() - 1)
    else:
        x = (torch.randint(-260, 261, (rows, cols), generator=g, device="cuda").double() * 2.0 ** -149).float()
    y = torch.zeros_like(x)
    tau = tao.tao_bound_norm(k, x, y, gamma, None, eps=0.0)
    assert torch.isfinite(tau).all()
    off = torch.exp2(-torch.randint(8, 15, x.shape, generator=g, device="cuda").double()) * (2.0 * torch.randint(0, 2, x.shape, generator=g, device="cuda") - 1)
    c = (tau.double() * (1 + off)).float()
    want = tao.tao_check_and_profile(c, y, tau)
    got = tao.tao_bound_check_norm(k, x, y, c, gamma, None, eps=0.0)
    for key in want:
        assert np.array_equal(np.asarray(got[key]), np.asarray(want[key])), key


def test_act_factor_below_the_normal_range(tao):
    n = 5 << 20
    g = torch.Generator(device="cuda").manual_seed(n)
    model = tao.FpModel(c_erf=1e-36)                         # c_erf u is a subnormal binary32 number
    x = 1e37 * (0.5 + torch.rand(n, generator=g, device="cuda"))
    y = torch.zeros_like(x)
    tau = tao.tao_bound_act(tao.ACT_GELU_ERF, x, y, model=model)
    off = torch.exp2(-torch.randint(8, 15, x.shape, generator=g, device="cuda").double()) * (2.0 * torch.randint(0, 2, x.shape, generator=g, device="cuda") - 1)
    c = (tau.double() * (1 + off)).float()
    want = tao.tao_check_and_profile(c, y, tau)
    got = tao.tao_bound_check_act(tao.ACT_GELU_ERF, x, y, c, model=model)
    for key in want:
        assert np.array_equal(np.asarray(got[key]), np.asarray(want[key])), key


def _padded(t, ld, offset):
    """The same values with a leading dimension beyond the row, `offset` floats into it; what lies between is NaN."""
    wide = torch.full((t.shape[0], ld), float("nan"), device=t.device)
    wide[:, offset:offset + t.shape[1]] = t
    return wide[:, offset:offset + t.shape[1]]


# rows with ld > cols on the quick routes: whole aligned vectors, padded; rows misaligned by 4 bytes; ragged rows
@pytest.mark.parametrize("kind", ["softmax", "layernorm", "rmsnorm"])
@pytest.mark.parametrize("rows,cols,ld,offset", [(16384, 128, 136, 0), (16384, 128, 132, 1), (16385, 511, 513, 0), (16390, 512, 520, 4), (8192, 768, 772, 0),
                                                 (8193, 1021, 1030, 2), (8192, 1024, 1028, 0), (16384, 1028, 1032, 0), (16384, 2048, 2052, 0),
                                                 (16385, 2048, 2053, 1), (4096, 4096, 4100, 0), (2048, 8190, 8193, 1)])
def test_strided_rows(tao, kind, rows, cols, ld, offset):
    g = torch.Generator(device="cuda").manual_seed(rows + cols + ld)
    x = torch.randn((rows, cols), generator=g, device="cuda")
    if kind == "softmax":
        x[::3, cols // 2:] = float("-inf")
        y = torch.softmax(x, -1)
        tau = tao.tao_bound_softmax(x, y)
    else:
        k = tao.NORM_LAYERNORM if kind == "layernorm" else tao.NORM_RMSNORM
        gamma = 1 + 0.1 * torch.randn(cols, generator=g, device="cuda")
        y = ((x - (x.mean(-1, keepdim=True) if kind == "layernorm" else 0)) * torch.rsqrt((x * x).mean(-1, keepdim=True) + 1e-5) * gamma)
        tau = tao.tao_bound_norm(k, x, y, gamma, None, eps=1e-5)
    # claims two output steps and more inside or outside the bound, so that a last-bit difference between the two kernels'
    # bounds (rows added in another order) cannot move one across it
    step = (torch.nextafter(y.abs(), torch.full_like(y, float("inf"))) - y.abs()).double()
    f = torch.randint(0, 8, y.shape, generator=g, device="cuda").double()
    t = tau.double()
    c = (y.double() + torch.where(f == 0, t + 2 * step, torch.where(f == 1, (t - 2 * step).clamp(min=0), t * (f - 4) / 4))).float()
    keep = (((c.double() - y.double()).abs() - t).abs() > 1e-6 * t) | (t == 0)
    c = torch.where(keep, c, y)
    want = tao.tao_check_and_profile(c, y, tau)
    assert want["violations"] > 0
    xs, ys, cs = (_padded(v, ld, offset) for v in (x, y, c))
    got = tao.tao_bound_check_softmax(xs, ys, cs) if kind == "softmax" else tao.tao_bound_check_norm(k, xs, ys, cs, gamma, None, eps=1e-5)
    for key in want:
        assert np.array_equal(np.asarray(got[key]), np.asarray(want[key])), key


@pytest.mark.parametrize("share", [0.0, 1e-5, 0.01])
@pytest.mark.parametrize("op", ["gelu", "silu", "softmax", "layernorm", "rmsnorm"])
def test_claims_that_equal_the_reference(tao, op, share):
    """All claims, or all but a few, equal to the re-executed values: no error is known for long, or ever."""
    rows, cols = 16384, 640
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn((rows, cols), generator=g, device="cuda")
    x[:, 3] = 0.0
    gamma = 1 + 0.1 * torch.randn(cols, generator=g, device="cuda")
    y = dict(gelu=lambda: torch.nn.functional.gelu(x), silu=lambda: torch.nn.functional.silu(x), softmax=lambda: torch.softmax(x, -1),
             layernorm=lambda: (x - x.mean(-1, keepdim=True)) * torch.rsqrt(x.var(-1, keepdim=True, unbiased=False) + 1e-5) * gamma,
             rmsnorm=lambda: x * torch.rsqrt((x * x).mean(-1, keepdim=True) + 1e-5) * gamma)[op]()
    c = torch.where(torch.rand(y.shape, generator=g, device="cuda") < share, y * (1 + 2.0 ** -12), y)
    y[5, 7] = c[5, 7] = float("inf"); y[6, 7] = c[6, 7] = float("nan")
    kind = dict(gelu=tao.ACT_GELU_ERF, silu=tao.ACT_SILU, layernorm=tao.NORM_LAYERNORM, rmsnorm=tao.NORM_RMSNORM).get(op)
    if op == "softmax":
        tau, got = tao.tao_bound_softmax(x, y), tao.tao_bound_check_softmax(x, y, c)
    elif op in ("gelu", "silu"):
        tau, got = tao.tao_bound_act(kind, x, y), tao.tao_bound_check_act(kind, x, y, c)
    else:
        tau, got = tao.tao_bound_norm(kind, x, y, gamma, None, eps=1e-5), tao.tao_bound_check_norm(kind, x, y, c, gamma, None, eps=1e-5)
    want = tao.tao_check_and_profile(c, y, tau)
    for key in want:
        a, b = np.asarray(got[key]), np.asarray(want[key])
        assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f"), key


# both sides of the rules by which one workgroup forms the profile itself, and the smallest tensors
@pytest.mark.parametrize("n", [1, 2, 3, 63, 64, 1025, 4097, 8192, 8193, 16384, 16385])
def test_small_tensors(tao, n):
    g = torch.Generator(device="cuda").manual_seed(n)
    x, x2 = torch.randn(n, generator=g, device="cuda"), torch.randn(n, generator=g, device="cuda")
    for kind, two in ((tao.ACT_GELU_ERF, False), (tao.ACT_SILU, False), (tao.ACT_MUL, True)):
        y = x * x2 if two else x / (1 + torch.exp(-x))
        tau = tao.tao_bound_act(kind, x, y, x2=x2 if two else None)
        c = _claims(y, tau, g)
        if n > 3:
            c[1], y[2], c[2] = float("nan"), 0.0, 0.0
        tau = tao.tao_bound_act(kind, x, y, x2=x2 if two else None)
        got = tao.tao_bound_check_act(kind, x, y, c, x2=x2 if two else None, eps_rel=0.0)
        streamed = tao.tao_check_and_profile(c, y, tau, eps_rel=0.0)
        want = oracle.check_and_profile(c.cpu().numpy(), y.cpu().numpy(), tau.cpu().numpy(), eps_rel=0.0)
        for key in streamed:
            a, b, w = np.asarray(got[key]), np.asarray(streamed[key]), np.asarray(want[key])
            assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f"), key
            assert np.array_equal(a, w.astype(a.dtype), equal_nan=a.dtype.kind == "f"), key


@pytest.mark.parametrize("rows,cols", [(1, 1), (1, 5), (4, 768), (8, 768), (9, 768), (16, 128), (33, 200), (1, 4096), (2, 4096), (3, 4096), (1, 9000), (2, 9000)])
def test_few_rows(tao, rows, cols):
    g = torch.Generator(device="cuda").manual_seed(rows + cols)
    x = torch.randn((rows, cols), generator=g, device="cuda")
    y = torch.softmax(x, -1)
    tau = tao.tao_bound_softmax(x, y)
    c = _claims(y, tau, g)
    want, got = tao.tao_check_and_profile(c, y, tau), tao.tao_bound_check_softmax(x, y, c)
    for key in want:
        a, b = np.asarray(got[key]), np.asarray(want[key])
        assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f"), key
