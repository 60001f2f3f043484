"""Checked products that the first slab of their reduction decides: a lower limit of every bound is enough for claims far inside, the others take
all products.  Claims that need them in some tiles, in all and in none, next to NaN claims and to comparisons left open, and operands beyond the
screen's range behind the first slab: every profile equals that of the stored bound and the streaming check, field for field."""
import pytest
import torch

from test_gpu_screen import _same, tao  # noqa: F401

pytestmark = pytest.mark.gpu

# Products by the form that checks them.  Few 64 x 64 tiles: reductions of more than twelve groups of 32 k, of three to five slabs and their remainders,
# tiles of one row and of one column.  128 x 128: a tile for a workgroup, two and three, with edges; whole slabs and remainders.
FEW, SHORT, LARGE, NARROW = "1, 1, 2, 2, 4, 2, 2, 0, true", "1, 1, 2, 2, 4, 2, 2, 0, false", "2, 2, 2, 2, 2, 2, 2, 0, true", "1, 2, 2, 2, 1, 3, 3, 0, false"
SHAPES = {FEW: [(1, 300, 200, 2080), (3, 65, 129, 385), (1, 65, 129, 416), (1, 192, 128, 417), (2, 257, 65, 448), (1, 130, 131, 512), (1, 1, 640, 500), (1, 640, 1, 640)],
          SHORT: [(3, 65, 129, 384), (1, 130, 131, 128)],
          LARGE: [(1, 2850, 3061, 300), (1, 4200, 4100, 264), (2, 2100, 2060, 1100), (1, 2050, 2052, 288), (1, 2100, 4004, 320)],
          NARROW: [(1, 2050, 2052, 256)]}
ALL_SHAPES = [shape for shapes in SHAPES.values() for shape in shapes]


def _claims(y, tau, g):
    """Claims by name: honest, then with errors of 0.3 and 1 times the bound in parts of the tensor, and NaN among them."""
    pick = torch.randint(-2, 3, y.shape, generator=g, device="cuda")
    honest = (y.double() * (1 + 2.0 ** -23 * pick)).float()
    inside, at = (y.double() + 0.3 * tau.double()).float(), (y.double() + tau.double()).float()
    u = torch.rand(y.shape, generator=g, device="cuda")
    rows = torch.arange(y.shape[-2], device="cuda")[:, None].expand(y.shape[-2:])
    last = torch.zeros_like(u, dtype=torch.bool)
    last.view(-1)[-1] = True
    return dict(honest=honest, inside=inside, last=torch.where(last, inside, honest), last_at=torch.where(last, at, honest),
                few=torch.where(u < 1e-4, inside, honest), some=torch.where(u < 0.02, inside, honest),
                first_rows=torch.where(rows < 64, inside, honest), later_rows=torch.where(rows >= 64, inside, honest),
                nan=torch.where(u < 1e-3, float("nan"), honest), nan_and_few=torch.where(u < 1e-3, float("nan"), torch.where(u > 0.999, inside, honest)),
                nan_and_at=torch.where(u < 1e-3, float("nan"), torch.where(u > 0.99, at, honest)),
                beyond=torch.where(u < 1e-3, (y.double() + 2 * tau.double()).float(), honest), infinite=torch.where(u < 1e-3, float("inf"), honest))


@pytest.mark.parametrize("batch,M,N,K", ALL_SHAPES)
def test_claims(tao, batch, M, N, K):  # noqa: F811
    g = torch.Generator(device="cuda").manual_seed(M + K)
    shape = (batch,) if batch > 1 else ()
    A, W = torch.randn((*shape, M, K), generator=g, device="cuda"), torch.randn((*shape, N, K), generator=g, device="cuda") * 0.02
    bias = torch.randn(N, generator=g, device="cuda") if M % 4 else None
    y = torch.matmul(A, W.transpose(-1, -2).contiguous()) + (0 if bias is None else bias)
    tau = tao.tao_bound_linear_split(A, W, bias)
    images = tao.tao_split_operand(A), tao.tao_split_operand(W)
    for kind, c in _claims(y, tau, g).items():
        want = tao.tao_check_and_profile(c, y, tau)
        _same(tao.tao_bound_check_linear(A, W, bias, y, c), want)
        _same(tao.tao_bound_check_linear_images(*images, M, N, K, y, c, bias=bias, batch=batch, shared_w=False), want)
    # a first slab of zeros decides nothing but errors of 0
    A[..., :160] = 0
    tau = tao.tao_bound_linear_split(A, W, bias)
    for c in (_claims(y, tau, g)["few"], y.clone()):
        _same(tao.tao_bound_check_linear(A, W, bias, y, c), tao.tao_check_and_profile(c, y, tau))


@pytest.mark.parametrize("B,H,C,Co,R,pad,st", [(11, 57, 96, 250, 1, 0, 1), (11, 56, 32, 256, 3, 1, 1), (22, 57, 32, 250, 3, 2, 1), (40, 57, 32, 300, 5, 0, 2), (11, 57, 64, 250, 1, 0, 1)])
def test_claims_of_a_convolution(tao, B, H, C, Co, R, pad, st):  # noqa: F811
    g = torch.Generator(device="cuda").manual_seed(B + H + Co)
    x = torch.randn((B, H, H, C), generator=g, device="cuda").abs()
    w = torch.randn((Co, R, R, C), generator=g, device="cuda") * 0.05
    tau = tao.tao_bound_conv2d_split(x, w, None, st, pad)
    y = torch.nn.functional.conv2d(x.permute(0, 3, 1, 2), w.permute(0, 3, 1, 2), None, st, pad).permute(0, 2, 3, 1).contiguous()
    for kind, c in _claims(y.view(-1, Co), tau.view(-1, Co), g).items():
        c = c.view(y.shape)
        _same(tao.tao_bound_check_conv2d(x, w, None, y, c, st, pad), tao.tao_check_and_profile(c, y, tau))
    for at, value in ((0, float("nan")), (x.numel() - 1, float("inf")), (x.numel() // 2 + C - 1, 2.0 ** 33)):
        x2 = x.clone()
        x2.view(-1)[at] = value
        tau = tao.tao_bound_conv2d_split(x2, w, None, st, pad)
        c = y * (1 + 2.0 ** -22)
        _same(tao.tao_bound_check_conv2d(x2, w, None, y, c, st, pad), tao.tao_check_and_profile(c, y, tau))


@pytest.mark.parametrize("M,N,K", [(300, 200, 2080), (2850, 3061, 300), (600, 9000, 1100), (1500, 700, 1500), (65, 129, 417)])
def test_operands_behind_the_first_slab(tao, M, N, K):  # noqa: F811
    g = torch.Generator(device="cuda").manual_seed(K)
    A0, W0 = torch.randn((M, K), generator=g, device="cuda"), torch.randn((N, K), generator=g, device="cuda")
    y = torch.matmul(A0, W0.t().contiguous())
    c = y * (1 + 2.0 ** -22)
    for i, value in enumerate((2.0 ** 32, 3e38, float("inf"), float("-inf"), float("nan"))):
        for row, k in ((-1, K - 1), (0, K - 1), (M // 2, 200)):
            A, W = A0.clone(), W0.clone()
            (W if (i + k) % 2 else A)[min(row, N - 1), k] = value
            _same(tao.tao_bound_check_linear(A, W, None, y, c), tao.tao_check_and_profile(c, y, tao.tao_bound_linear_split(A, W)))


def test_parts_of_a_batch_as_images(tao):  # noqa: F811
    """An image of a batch is passed on from one of its entries: what lies where a single image says whether it is ordinary are pieces then."""
    g = torch.Generator(device="cuda").manual_seed(3)
    B, M, N, K = 3, 256, 200, 2080
    A, W = torch.randn((B, M, K), generator=g, device="cuda"), torch.randn((N, K), generator=g, device="cuda")
    A[1, 5, K - 1] = float("nan")
    A[2, :8, :32] = 0
    image, w_image = tao.tao_split_operand(A), tao.tao_split_operand(W)
    one = (K // 32) * (M // 128) * 3 * 128 * 64
    for z in range(B):
        y = torch.matmul(A[z], W.t().contiguous()).nan_to_num(0.0)
        c = y * (1 + 2.0 ** -22)
        got = tao.tao_bound_check_linear_images(image[z * one:], w_image, M, N, K, y, c)
        _same(got, tao.tao_check_and_profile(c, y, tao.tao_bound_linear_split(A[z], W)))


def test_more_tiles_than_are_tried(tao):  # noqa: F811
    """A workgroup tries 256 tiles by their first slabs: the others take all products."""
    g = torch.Generator(device="cuda").manual_seed(4)
    n = 128 * 364                                            # 132496 tiles on 512 places
    A, W = torch.randn((n, 288), generator=g, device="cuda"), torch.randn((n, 288), generator=g, device="cuda")
    y = torch.full((n, n), 1.0, device="cuda")
    c = y.clone()
    c[::1000] *= 1 + 2.0 ** -20
    tau = tao.tao_bound_linear_split(A, W)
    c[0, 7], c[-1, -1] = 1 + 0.4 * tau[0, 7], 1 + 1.5 * tau[-1, -1]
    _same(tao.tao_bound_check_linear(A, W, None, y, c), tao.tao_check_and_profile(c, y, tau))
