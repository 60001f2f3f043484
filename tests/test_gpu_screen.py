"""The screen of the checked matmul bounds (one BF16 product decides the comparisons, the exact route does the rest): every profile
equals that of the stored bound and the streaming check, field for field, for claims that the screen settles and for claims that
it must leave alone, at the edges of its tiles, with operands outside its range, and in graph replays."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tao():
    import paper_2510_16028_amd as t
    t.lib()
    assert torch.cuda.is_available()
    return t


def _same(got, want):
    assert set(got) == set(want)
    for key in want:
        a, b = np.asarray(got[key]), np.asarray(want[key])
        assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f"), (key, got[key], want[key])


def _claim(kind, y, tau, g):
    yd, td = y.double(), tau.double()
    pick = torch.randint(0, 6, y.shape, generator=g, device=y.device)
    if kind == "honest":
        return (yd * (1 + 2.0 ** -23 * (pick - 2))).float()
    if kind == "equal":
        return y.clone()
    if kind == "far":                                        # inside and outside, none within a per cent of the bound
        f = torch.tensor([0.0, 0.5, 0.98, 1.02, -1.02, 3.0], dtype=torch.float64, device=y.device)
        return (yd + f[pick] * td).float()
    if kind == "near":
        return (yd + (1 + 2e-3 * torch.randn(y.shape, generator=g, device=y.device, dtype=torch.float64)) * td).float()
    c = (yd * (1 + 2.0 ** -23 * (pick - 2))).float()
    at = c.view(-1)
    n = at.numel()
    if kind == "one at its bound":
        at[n // 2] = (yd + td).float().view(-1)[n // 2]
    elif kind == "one beyond":
        at[n - 1] = (yd + 1.5 * td).float().view(-1)[n - 1] + 1e-30
    else:                                                    # values that no estimate settles
        at[0] = float("nan"); at[n // 3] = float("inf"); at[n // 2] = 3e38; at[n - 1] = -3e38
    return c


KINDS = ["honest", "equal", "far", "near", "one at its bound", "one beyond", "values"]
# both sides of the tile shapes and of the rules between them (128 x 128, 64 x 128, 64 x 64 with four and eight stages, A read as rows),
# remainders in every direction, groups of 32 k fewer than the stages and more, reductions in parts and not
SHAPES = [(1, 1, 1, 1), (1, 64, 64, 32), (1, 65, 63, 31), (3, 127, 129, 33), (1, 129, 130, 224), (1, 130, 131, 288), (1, 700, 66, 1100),
          (1, 2048, 2052, 64), (1, 2047, 2049, 264), (1, 2050, 2052, 300), (1, 1111, 3001, 1001), (2, 1500, 1500, 96), (5, 1000, 64, 160),
          (1, 33000, 128, 1056), (1, 33001, 100, 1088), (1, 16500, 250, 1056), (1, 300, 200, 4096), (1, 1024, 1024, 2080), (12, 512, 512, 64),
          (3, 200, 70, 96), (12, 512, 64, 512), (4, 300, 250, 4128), (17, 1000, 128, 64)]


@pytest.mark.parametrize("batch,M,N,K", SHAPES)
def test_profile_equals_bound_and_check(tao, batch, M, N, K):
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    shape = (batch,) if batch > 1 else ()
    A = torch.randn((*shape, M, K), generator=g, device="cuda")
    W = torch.randn((*shape, N, K), generator=g, device="cuda") * 0.02
    bias = torch.randn(N, generator=g, device="cuda") if (M + N) % 2 else None
    y = torch.matmul(A, W.transpose(-1, -2).contiguous()) + (0 if bias is None else bias)
    tau = tao.tao_bound_linear_split(A, W, bias)
    images = tao.tao_split_operand(A), tao.tao_split_operand(W)
    Wt = W.transpose(-1, -2).contiguous()
    for kind in KINDS:
        c = _claim(kind, y, tau, g)
        alpha, eps = (2.0, 0.0) if kind == "far" and M % 2 else (1.0, 1e-12)
        want = tao.tao_check_and_profile(c, y, tau, alpha=alpha, eps_rel=eps)
        _same(tao.tao_bound_check_linear(A, W, bias, y, c, alpha=alpha, eps_rel=eps), want)
        _same(tao.tao_bound_check_linear(A, Wt, bias, y, c, trans_w=True, alpha=alpha, eps_rel=eps), want)
        _same(tao.tao_bound_check_linear_images(*images, M, N, K, y, c, bias=bias, batch=batch, shared_w=False, alpha=alpha, eps_rel=eps), want)


@pytest.mark.parametrize("M,N,K", [(70, 70, 96), (256, 200, 96), (2100, 2060, 64), (33000, 100, 1056)])
def test_operands_outside_the_range(tao, M, N, K):
    """A large, infinite or NaN operand at any place decides nothing by the screen, nor do sums near the end of the subnormals."""
    g = torch.Generator(device="cuda").manual_seed(K)
    A0 = torch.rand((M, K), generator=g, device="cuda") + 0.5
    W0 = torch.rand((N, K), generator=g, device="cuda") + 0.5
    places = [0, 1, 5, 10, 15, 16, 23, 31, 32, K - 1]
    for i, k in enumerate(places):
        for value in (2.0 ** 32, 3e38, float("inf"), float("nan"))[i % 4:][:2]:
            A, W = A0.clone(), W0.clone()
            (A if i % 2 else W)[(0, M - 1)[i % 3 == 0] if i % 2 else (N - 1, 0)[i % 3 == 0], k] = value
            tau = tao.tao_bound_linear_split(A, W)
            y = torch.zeros((M, N), device="cuda")
            c = torch.full_like(y, 3e38); c[::2] = 1e-5
            _same(tao.tao_bound_check_linear(A, W, None, y, c), tao.tao_check_and_profile(c, y, tau))
    for sa, sw in ((2.0 ** -70, 2.0 ** -70), (2.0 ** -130, 2.0 ** 31), (2.0 ** -45, 2.0 ** -45), (0.0, 1.0)):
        A, W = A0 * sa, W0 * sw
        tau = tao.tao_bound_linear_split(A, W)
        y = tau * torch.rand((M, N), generator=g, device="cuda")
        c = (tau.double() * 1.9 * torch.rand((M, N), generator=g, device="cuda", dtype=torch.float64) + y.double()).float()
        _same(tao.tao_bound_check_linear(A, W, None, y, c), tao.tao_check_and_profile(c, y, tau))


@pytest.mark.parametrize("alpha,flags,u", [(0.0, 0, 2.0 ** -24), (1e-13, 0, 2.0 ** -24), (1e9, 0, 2.0 ** -24), (1.0, 1, 2.0 ** -24), (1.0, 0, 2.0 ** -11), (3.0, 0, 2.0 ** -30)])
def test_factors_and_models(tao, alpha, flags, u):
    g = torch.Generator(device="cuda").manual_seed(3)
    M, N, K = 300, 260, 160
    model = tao.FpModel(flags=flags, u=u)
    A, W = torch.randn((M, K), generator=g, device="cuda"), torch.randn((N, K), generator=g, device="cuda")
    bias = torch.randn(N, generator=g, device="cuda")
    bias[7], bias[9] = 1e30, float("inf")
    y = torch.matmul(A, W.t().contiguous())
    for b in (None, bias):
        tau = tao.tao_bound_linear_split(A, W, b, model=model)
        f = torch.rand((M, N), generator=g, device="cuda", dtype=torch.float64) * 2
        c = (y.double() + f * (alpha if alpha else 1.0) * tau.double().clamp(max=1e30)).float()
        _same(tao.tao_bound_check_linear(A, W, b, y, c, alpha=alpha, model=model), tao.tao_check_and_profile(c, y, tau, alpha=alpha))


@pytest.mark.parametrize("ldy,shift", [(260, 0), (264, 0), (261, 0), (260, 1)])
def test_padded_and_misaligned_rows(tao, ldy, shift):
    g = torch.Generator(device="cuda").manual_seed(ldy)
    M, N, K = 333, 260, 200
    A, W = torch.randn((M, K), generator=g, device="cuda"), torch.randn((N, K), generator=g, device="cuda")
    y = torch.matmul(A, W.t().contiguous())
    tau = tao.tao_bound_linear_split(A, W)
    ws = torch.empty(tao.tao_bound_check_linear_workspace_bytes(M, N, K), dtype=torch.uint8, device="cuda")
    for kind in ("far", "near"):
        c = _claim(kind, y, tau, g)
        pad = torch.full((2, M * ldy + 4), 7.0, device="cuda")
        rows = [p[shift:shift + M * ldy].view(M, ldy) for p in pad]
        rows[0][:, :N], rows[1][:, :N] = y, c
        out = tao.new_profile_buffer(A.device)
        rc = tao.lib().tao_bound_check_linear(A.data_ptr(), W.data_ptr(), None, rows[0].data_ptr(), rows[1].data_ptr(), None, M, N, K, K, K, ldy, 0,
                                              1, 0, 0, 0, 1.0, 1e-12, None, out.data_ptr(), ws.data_ptr(), ws.numel(),
                                              torch.cuda.current_stream().cuda_stream)
        assert rc == tao.OK
        _same(tao.read_profile(out), tao.tao_check_and_profile(c, y, tau))


# (batch, size, C, Cout, filter, stride, padding, dilation): tiles of 128 and of 64 columns, taps in the padding, a row tile's remainder
@pytest.mark.parametrize("B,H,C,Co,R,st,pad,dil", [(32, 28, 128, 512, 1, 1, 0, 1), (32, 57, 64, 96, 3, 2, 1, 1), (33, 40, 32, 64, 3, 1, 2, 2),
                                                   (30, 30, 96, 100, 3, 1, 1, 1), (9, 62, 32, 130, 5, 1, 2, 1)])
def test_convolution(tao, B, H, C, Co, R, st, pad, dil):
    g = torch.Generator(device="cuda").manual_seed(H)
    x = torch.randn((B, H, H, C), generator=g, device="cuda").abs()
    w = torch.randn((Co, R, R, C), generator=g, device="cuda") * 0.05
    bias = torch.randn(Co, generator=g, device="cuda") if Co % 4 == 0 else None
    assert tao.tao_conv2d_split_supported(tuple(x.shape), tuple(w.shape), st, pad, dil)
    for large in (False, True):
        if large:
            x[B - 1, H // 2, H // 2, C - 1] = 1e35
        tau = tao.tao_bound_conv2d_split(x, w, bias, st, pad, dil)
        y = torch.nn.functional.conv2d(x.permute(0, 3, 1, 2), w.permute(0, 3, 1, 2), bias, st, pad, dil).permute(0, 2, 3, 1).contiguous()
        geom = (B, H, H, C, Co, R, R, st, st, pad, pad, dil, dil)
        full = int(tao.lib().tao_conv2d_split_workspace_bytes(*geom, 1))
        small = full - (B * H * H * C * 2 + 64)              # what the exact route alone needs is still enough
        for kind in ("honest", "far", "near"):
            c = _claim(kind, y, tau, g)
            want = tao.tao_check_and_profile(c, y, tau)
            for n in (full, small):
                ws = torch.empty(n, dtype=torch.uint8, device="cuda")
                _same(tao.tao_bound_check_conv2d(x, w, bias, y, c, st, pad, dil, ws=ws), want)


# An error of which a binary32 estimate leaves 0, though claim and output differ: the quotient is a half of the smallest subnormal and a
# little more, and rounds up to it; the estimate, whose denominator is rounded to the next even binary32 value, comes down to a tie and rounds
# to 0.  unit: half the denominator, times 2^-149 (for the smaller ones as a binary32 value's bits).
@pytest.mark.parametrize("eps,unit", [(2 - 2.0 ** -40, 2.0 ** -149), (6 - 2.0 ** -40, 3 * 2.0 ** -149), (2.0 ** 40 - 1, 2.0 ** -110), (1.0, 2.0 ** -149)])
@pytest.mark.parametrize("batch,M,N,K", [(1, 300, 260, 100), (1, 2085, 3205, 100), (1, 2850, 3061, 300), (1, 16500, 130, 64)])
def test_estimates_that_underflow(tao, batch, M, N, K, eps, unit):
    g = torch.Generator(device="cuda").manual_seed(M)
    A, W = torch.randn((M, K), generator=g, device="cuda"), torch.randn((N, K), generator=g, device="cuda")
    y, tau = torch.zeros((M, N), device="cuda"), tao.tao_bound_linear_split(A, W)
    bits = int(np.float32(unit).view(np.int32))
    for share in (0.5, 1e-3):                                # (the others are errors of 0)
        c = ((torch.rand((M, N), generator=g, device="cuda") < share).to(torch.int32) * bits).view(torch.float32)
        want = tao.tao_check_and_profile(c, y, tau, eps_rel=eps)
        assert want["max_rel"] == 2.0 ** -149, want["max_rel"]
        _same(tao.tao_bound_check_linear(A, W, None, y, c, eps_rel=eps), want)


def test_estimates_that_underflow_in_a_convolution(tao):
    g = torch.Generator(device="cuda").manual_seed(7)
    x, w = torch.randn((11, 57, 57, 32), generator=g, device="cuda"), torch.randn((250, 1, 1, 32), generator=g, device="cuda")
    tau = tao.tao_bound_conv2d_split(x, w)
    y, eps = torch.zeros_like(tau), 2 - 2.0 ** -40
    c = (torch.rand(tau.shape, generator=g, device="cuda") < 0.5).to(torch.int32).view(torch.float32)
    want = tao.tao_check_and_profile(c, y, tau, eps_rel=eps)
    assert want["max_rel"] == 2.0 ** -149, want["max_rel"]
    _same(tao.tao_bound_check_conv2d(x, w, None, y, c, eps_rel=eps), want)


def test_replays_on_claims_of_either_kind(tao):
    g = torch.Generator(device="cuda").manual_seed(1)
    M, N, K = 520, 1030, 200
    A, W = torch.randn((M, K), generator=g, device="cuda"), torch.randn((N, K), generator=g, device="cuda")
    y = torch.matmul(A, W.t().contiguous())
    tau = tao.tao_bound_linear_split(A, W)
    images = tao.tao_split_operand(A), tao.tao_split_operand(W)
    c = y.clone()
    ws = torch.empty(tao.tao_bound_check_linear_workspace_bytes(M, N, K), dtype=torch.uint8, device="cuda")
    wi = torch.empty(tao.lib().tao_check_linear_images_workspace_bytes(M, N, K, 1), dtype=torch.uint8, device="cuda")
    outs = [tao.new_profile_buffer(A.device) for _ in range(2)]

    def step():
        tao.tao_bound_check_linear(A, W, None, y, c, out=outs[0], ws=ws, readback=False)
        tao.tao_bound_check_linear_images(*images, M, N, K, y, c, out=outs[1], ws=wi, readback=False)

    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for kind in ("honest", "near", "far", "near", "equal", "values", "honest"):
        c.copy_(_claim(kind, y, tau, g))
        want = tao.tao_check_and_profile(c, y, tau)
        graph.replay()
        torch.cuda.synchronize()
        for o in outs:
            _same(tao.read_profile(o), want)
