"""Tiles that a workgroup walks: the next tile's claims and outputs are requested while the one before is checked.  More tiles than workgroups
that fit the chip at once, in each form of the left operand, with edges among a workgroup's tiles, errors of 0
alone, among others and not at all: every profile equals that of the stored bound and the streaming check, field for field."""
import pytest
import torch

from test_gpu_screen import _claim, _same, tao  # noqa: F401

pytestmark = pytest.mark.gpu


# 64 x 128 tiles (33 x 26 and 3 x 17 x 17 on 768 places, 66 x 26: a first, a middle and a last tile for a workgroup), 128 x 128 (23 x 24 on
# 512, K a whole number of stages and not; 33 x 33), rows (1032 and 1025 tiles on 512)
@pytest.mark.parametrize("batch,M,N,K", [(1, 2085, 3205, 100), (3, 1069, 2060, 33), (1, 4200, 3205, 100), (1, 2850, 3061, 300), (1, 2944, 3072, 320),
                                         (1, 4200, 4100, 264), (1, 33005, 130, 64), (1, 65600, 128, 96)])
def test_walked_tiles(tao, batch, M, N, K):  # noqa: F811
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    shape = (batch,) if batch > 1 else ()
    A = torch.randn((*shape, M, K), generator=g, device="cuda")
    W = torch.randn((*shape, N, K), generator=g, device="cuda") * 0.02
    y = torch.matmul(A, W.transpose(-1, -2).contiguous())
    tau = tao.tao_bound_linear_split(A, W, None)
    for kind in ("honest", "equal", "far", "values"):
        c = _claim(kind, y, tau, g)
        want = tao.tao_check_and_profile(c, y, tau)
        _same(tao.tao_bound_check_linear(A, W, None, y, c), want)


# 128 x 128 tiles on 512 places: 280 x 2 and 270 x 2, and 559 x 2
@pytest.mark.parametrize("B,H,C,Co,R,pad", [(11, 57, 32, 250, 1, 0), (11, 56, 32, 256, 3, 1), (22, 57, 32, 250, 3, 1)])
def test_walked_tiles_of_a_convolution(tao, B, H, C, Co, R, pad):  # noqa: F811
    g = torch.Generator(device="cuda").manual_seed(B + H + Co)
    x = torch.randn((B, H, H, C), generator=g, device="cuda")
    w = torch.randn((Co, R, R, C), generator=g, device="cuda") * 0.05
    tau = tao.tao_bound_conv2d_split(x, w, None, 1, pad)
    y = torch.randn(tau.shape, generator=g, device="cuda") * tau.mean() * 1e3      # (the check does not ask where outputs come from)
    for kind in ("honest", "equal", "far", "values"):
        c = _claim(kind, y, tau, g)
        _same(tao.tao_bound_check_conv2d(x, w, None, y, c, 1, pad), tao.tao_check_and_profile(c, y, tau))


# operands beyond what is screened: nothing is decided, all wavefronts of a workgroup stop forming products at the same tile (they meet at
# fewer barriers from there on), and every error's bin still counts.  Workgroups of three tiles and of two in each form; of one, where none stop
@pytest.mark.parametrize("M,N,K", [(4200, 4100, 64), (3300, 3300, 64), (4200, 4100, 264), (2850, 3061, 300), (33005, 130, 64), (2300, 2050, 64)])
def test_walked_tiles_without_products(tao, M, N, K):  # noqa: F811
    g = torch.Generator(device="cuda").manual_seed(M + N)
    A = torch.randn((M, K), generator=g, device="cuda") * 2.0 ** 40
    W = torch.randn((N, K), generator=g, device="cuda")
    y = torch.matmul(A, W.t().contiguous())
    c = _claim("honest", y, y, g)
    c[::2] = y[::2] * 1.5
    want = tao.tao_check_and_profile(c, y, tao.tao_bound_linear_split(A, W, None))
    for _ in range(3):
        _same(tao.tao_bound_check_linear(A, W, None, y, c), want)


# Claims that equal the outputs but for a few elements: workgroups meet their first error late, in one lane or a few, and go on to tiles at which
# some of their lanes know of an error and the others do not.  The largest is met after smaller ones, before them, alone.  (A bias whose bits
# are larger than any error's: none may pass for one.)
@pytest.mark.parametrize("batch,M,N,K", [(1, 2085, 3205, 100), (1, 4200, 3205, 33), (1, 2850, 3061, 300), (1, 33005, 130, 64)])
def test_walked_tiles_with_few_errors(tao, batch, M, N, K):  # noqa: F811
    g = torch.Generator(device="cuda").manual_seed(M * 3 + K)
    A, W = torch.randn((M, K), generator=g, device="cuda"), torch.randn((N, K), generator=g, device="cuda")
    y = torch.rand((M, N), generator=g, device="cuda") + 1
    bias = torch.full((N,), 1e6, device="cuda")
    tau = tao.tao_bound_linear_split(A, W, bias)
    for few, kind in ((1, "one"), (30, "growing"), (700, "growing"), (700, "shrinking"), (7000, "growing")):
        c = y.clone()
        at = torch.randint(0, M * N, (few,), generator=g, device="cuda").sort().values
        # (relative errors over 2^-22 .. 2^-4, along the walk)
        size = torch.linspace(-22, -4, few, device="cuda") if few > 1 else torch.tensor([-12.0], device="cuda")
        if kind == "shrinking":
            size = size.flip(0)
        c.view(-1)[at] = y.view(-1)[at] * (1 + torch.exp2(size))
        _same(tao.tao_bound_check_linear(A, W, bias, y, c), tao.tao_check_and_profile(c, y, tau))


# both ways of telling an error of 0, and the line between them, in each larger form
@pytest.mark.parametrize("eps", [1.0, 1.0000000000000002, 3.0])
@pytest.mark.parametrize("M,N,K", [(2085, 3205, 100), (2850, 3061, 300), (33005, 130, 64)])
def test_walked_tiles_with_large_denominators(tao, M, N, K, eps):  # noqa: F811
    g = torch.Generator(device="cuda").manual_seed(M + K)
    A, W = torch.randn((M, K), generator=g, device="cuda"), torch.randn((N, K), generator=g, device="cuda") * 0.02
    y = torch.matmul(A, W.t().contiguous())
    tau = tao.tao_bound_linear_split(A, W, None)
    for kind in ("honest", "equal", "far", "values"):
        c = _claim(kind, y, tau, g)
        _same(tao.tao_bound_check_linear(A, W, None, y, c, eps_rel=eps), tao.tao_check_and_profile(c, y, tau, eps_rel=eps))


def test_walked_convolution_with_large_denominators(tao):  # noqa: F811
    g = torch.Generator(device="cuda").manual_seed(2)
    x, w = torch.randn((11, 57, 57, 32), generator=g, device="cuda"), torch.randn((250, 1, 1, 32), generator=g, device="cuda") * 0.05
    tau = tao.tao_bound_conv2d_split(x, w)
    y = torch.randn(tau.shape, generator=g, device="cuda") * tau.mean() * 1e3
    for kind in ("honest", "equal", "far", "values"):
        c = _claim(kind, y, tau, g)
        _same(tao.tao_bound_check_conv2d(x, w, None, y, c, eps_rel=3.0), tao.tao_check_and_profile(c, y, tau, eps_rel=3.0))
