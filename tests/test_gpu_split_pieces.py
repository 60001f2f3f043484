"""The BF16-split matmul bound on operands at the edges of its three pieces: halfway remainders, the top of the binary32
range, operands below 2^-110 (whose last piece leaves BF16's grid) and subnormal ones, infinities and NaN."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


@pytest.fixture(scope="module")
def tao():
    import paper_2510_16028_amd as t
    t.lib()
    assert torch.cuda.is_available()
    return t


def _operand(rng, rows, K, kind):
    sign = np.where(rng.random((rows, K)) < 0.5, -1.0, 1.0)
    man = rng.integers(0, 1 << 23, (rows, K))
    if kind == "halves":                                     # remainders of half a step, one unit to either side
        man = (rng.integers(0, 128, (rows, K)) << 16) | (0x8000 + rng.integers(-1, 2, (rows, K)))
        man = np.where(rng.random((rows, K)) < 0.5, man, (1 << 15) - (1 << 14) - (1 << 6) + rng.integers(0, 2, (rows, K)))
        e = rng.integers(-3, 4, (rows, K))
    elif kind == "top":
        man = np.where(rng.random((rows, K)) < 0.5, man, (1 << 23) - 1 - rng.integers(0, 1 << 15, (rows, K)))
        e = np.full((rows, K), 127)
    elif kind == "small":
        e = rng.integers(-126, -104, (rows, K))
    elif kind == "subnormal":
        return (sign * rng.integers(0, 1 << 23, (rows, K)) * 2.0 ** -149).astype(np.float32)
    else:
        e = rng.integers(-2, 3, (rows, K))
    return (sign * np.ldexp(((1 << 23) + man).astype(np.float64), e - 23)).astype(np.float32)


# relative room above the exact bound: 1e-6, and what the raised last piece adds to operands below 2^-110:
# at most two steps of 2^-133 relative to 2^-126 (normal) -- subnormal ones are bounded from below only
@pytest.mark.parametrize("a,w,scale,room", [
    ("plain", "plain", 0, 1e-6), ("halves", "halves", 0, 1e-6), ("top", "plain", -60, 1e-6), ("plain", "top", -60, 1e-6),
    ("small", "halves", 60, 1e-6 + 2.0 ** -6), ("halves", "small", 60, 1e-6 + 2.0 ** -6), ("subnormal", "halves", 60, None),
])
@pytest.mark.parametrize("M,N,K", [(5, 3, 33), (130, 200, 160)])
def test_bound_at_the_edges_of_the_pieces(tao, a, w, scale, room, M, N, K):
    rng = np.random.Generator(np.random.Philox(M + K + len(a)))
    A, W = _operand(rng, M, K, a), _operand(rng, N, K, w)
    if scale > 0:                                            # products well inside the normal range
        A, W = (A, (W * 2.0 ** scale).astype(np.float32)) if a in ("small", "subnormal") else ((A * 2.0 ** scale).astype(np.float32), W)
    elif scale < 0:
        A, W = (A, (W * 2.0 ** scale).astype(np.float32)) if a == "top" else ((A * 2.0 ** scale).astype(np.float32), W)
    tau = tao.tao_bound_linear_split(torch.from_numpy(A).cuda(), torch.from_numpy(W).cuda()).cpu().numpy().astype(np.float64)
    # products of two binary32 values are exact in binary64; K additions of them stay within K 2^-53
    exact = np.abs(A.astype(np.float64)) @ np.abs(W.astype(np.float64)).T * (K * U / (1 - K * U))
    slack = (K + 8) * 2.0 ** -53
    assert np.isfinite(tau).all()
    assert (tau >= exact * (1 - slack)).all()
    if room is not None:
        assert (tau <= exact * (1 + room) * (1 + slack)).all()


@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan"), "payload"])
def test_non_finite_operands_never_give_a_finite_bound(tao, bad):
    g = torch.Generator().manual_seed(3)
    A, W = torch.randn((40, 96), generator=g), torch.randn((24, 96), generator=g)
    if bad == "payload":                                     # NaN patterns at both ends of the payload
        A.view(torch.int32)[7, 50] = 0x7f800001
        A.view(torch.int32)[8, 51] = 0x7fffffff
        W.view(torch.int32)[3, 60] = -1
    else:
        A[7, 50] = bad; A[8, 51] = bad; W[3, 60] = bad
    W[5] = 0.0                                               # inf x 0 as well
    tau = tao.tao_bound_linear_split(A.cuda(), W.cuda()).cpu()
    hit = torch.zeros(40, 24, dtype=torch.bool)
    hit[7], hit[8], hit[:, 3] = True, True, True
    assert not torch.isfinite(tau[hit]).any() and torch.isfinite(tau[~hit]).all()


def _overflowing(rng, M, N, K, what):
    """Finite operands whose products, or their sums, leave the binary32 range or stay just below its end."""
    A = rng.uniform(0.5, 1.0, (M, K)).astype(np.float32)
    W = rng.uniform(0.5, 1.0, (N, K)).astype(np.float32)
    if what == "products":                                   # every product is beyond 2^128; pieces with a negative middle one
        A, W = (1.998 * 2.0 ** 70 * np.sign(A)).astype(np.float32), (2.0 ** 70 * np.sign(W)).astype(np.float32)
    elif what == "some":                                     # a few products of some rows
        A[::3, 5::32] = 1.998 * 2.0 ** 70
        W[::2, 5::32] = 2.0 ** 66
    else:                                                    # sums of 16 products 2^128 (1 - 2^-8): each hi piece is rounded up to 2^62
        A[:] = np.float32((1.0 - 0.49 * 2.0 ** -8) * 2.0 ** 62)
        W[:] = A[0, 0]
    return A * rng.choice([-1.0, 1.0], A.shape).astype(np.float32), W


# the routes of the BF16 scheme: parts, one workgroup per tile, A cut while it is loaded, the walk over tiles; bound and check
@pytest.mark.parametrize("M,N,K", [(130, 200, 96), (256, 256, 1088), (4200, 4100, 64), (2100, 2060, 1088), (33000, 128, 1056)])
@pytest.mark.parametrize("what", ["products", "some", "sums"])
def test_finite_operands_beyond_the_range(tao, M, N, K, what):
    rng = np.random.Generator(np.random.Philox(M + K))
    A, W = _overflowing(rng, M, N, K, what)
    a, w = torch.from_numpy(A).cuda(), torch.from_numpy(W).cuda()
    tau = tao.tao_bound_linear_split(a, w)
    # (torch's binary64 product: K additions within K 2^-53)
    exact = torch.matmul(a.double().abs(), w.double().abs().t().contiguous()) * (K * U / (1 - K * U))
    slack = (K + 8) * 2.0 ** -53
    assert not torch.isnan(tau).any()
    assert (tau.double() >= exact * (1 - slack)).all()
    assert (tau.double() <= exact * (1 + 1e-6) * (1 + slack))[exact * (1 + 1e-6) < 2.0 ** 128].all()
    y = torch.zeros_like(tau)
    c = torch.full_like(tau, 3e38)
    c[::2] = 1.0
    want = tao.tao_check_and_profile(c, y, tau)
    for got in (tao.tao_bound_check_linear(a, w, None, y, c), tao.tao_bound_check_linear(a, w, None, y, c, model=tao.FpModel(flags=tao.FLAG_CHECK_IN_EPILOGUE))):
        for key in want:
            assert np.array_equal(np.asarray(got[key]), np.asarray(want[key])), key
    images = tao.tao_split_operand(a), tao.tao_split_operand(w)
    assert torch.equal(tao.tao_bound_linear_images(*images, M, N, K), tau)


def test_conv_of_finite_operands_beyond_the_range(tao):
    rng = np.random.Generator(np.random.Philox(5))
    x = np.abs(rng.standard_normal((32, 34, 34, 32))).astype(np.float32)
    w = rng.standard_normal((128, 3, 3, 32)).astype(np.float32)
    x[3, 4:9, 7, 11] = 1.998 * 2.0 ** 70
    w[5, 1, 1, 11] = 2.0 ** 70
    x, w = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    assert tao.tao_conv2d_split_supported(tuple(x.shape), tuple(w.shape), 1, 1, 1)
    tau = tao.tao_bound_conv2d_split(x, w, None, 1, 1)
    cols = torch.nn.functional.unfold(x.double().permute(0, 3, 1, 2), 3, padding=1)           # [batch][C R S][positions]
    K = 288
    exact = torch.matmul(cols.transpose(1, 2).contiguous(), w.double().abs().permute(0, 3, 1, 2).reshape(128, -1).t().contiguous())
    exact = (exact * (K * U / (1 - K * U))).reshape(tau.shape)
    slack = (K + 8) * 2.0 ** -53
    assert not torch.isnan(tau).any()
    assert (tau.double() >= exact * (1 - slack)).all()
    assert (tau.double() <= exact * (1 + 1e-6) * (1 + slack))[exact * (1 + 1e-6) < 2.0 ** 128].all()


@pytest.mark.parametrize("rows", [1, 3, 4, 13, 16, 17])
@pytest.mark.parametrize("batch,K", [(1, 511 * 32), (1, 512 * 32 + 5), (3, 6000), (600, 9), (1, 33)])
def test_images_of_few_rows(tao, rows, batch, K):
    """The image of a few rows, cut by workgroups or by wavefronts, is what the same rows have in the image of more (the layout does not depend on
    the number of rows up to 128): every piece of every row that exists, and zeros up to a multiple of four rows and of 32 k."""
    g = torch.Generator(device="cuda").manual_seed(rows + K)
    few = torch.randn((batch, rows, K), generator=g, device="cuda")
    more = torch.zeros((batch, 40, K), device="cuda")
    more[:, :rows] = few
    images = []
    for x in (few, more):
        out = torch.full((tao.tao_split_image_bytes(x.shape[1], K, batch),), 0x5a, dtype=torch.uint8, device="cuda")
        n = batch * ((K + 31) // 32) * 3 * 128 * 64
        images.append(tao.tao_split_operand(x, out=out)[:n].view(-1, 128, 64)[:, :(rows + 3) // 4 * 4])
    assert torch.equal(*images)


# units of 64 rows x 32 k: a workgroup of one, two, three and four parts, some units to spare, and walks of two to five rounds of whole units and of cut ones
@pytest.mark.parametrize("rows,K,batch,trans", [(1000, 1001, 1, False), (1100, 1000, 1, False), (1500, 1500, 1, False), (1500, 1500, 1, True), (960, 1920, 2, False), (2176, 2056, 1, False),
                                                (2100, 2056, 1, False), (2049, 2056, 1, False), (2052, 2056, 2, False), (2176, 2055, 1, False), (2176, 2056, 1, True), (4352, 4096, 1, False), (320, 40, 450, False), (320, 260, 100, False), (15, 2300 * 32, 1, False), (8, 8300 * 32, 1, False)])
def test_images_of_many_units(tao, rows, K, batch, trans):
    """Every element's pieces add up to it, whichever part of a workgroup has cut it, and each large one is told by the marks behind the image where a product can read them."""
    g = torch.Generator(device="cuda").manual_seed(rows + K)
    x = torch.randn((batch, rows, K), generator=g, device="cuda")
    groups, blocks = (K + 31) // 32, (rows + 127) // 128
    size = batch * groups * blocks * 3 * 128 * 64
    r, k = torch.arange(128, device="cuda"), torch.arange(32, device="cuda")
    at = ((k[None] // 8) ^ ((r[:, None] >> 2) & 3)) * 8 + k[None] % 8
    for where in (None, (0, 0, 0), (-1, -1, -1), (batch // 2, rows // 2, K // 3)):
        if where:
            x[where] = -2.0 ** 33
        out = torch.full((tao.tao_split_image_bytes(rows, K, batch),), 0x5a, dtype=torch.uint8, device="cuda")
        src = x.transpose(1, 2).contiguous() if trans else x
        tao.tao_split_operand(src if batch > 1 else src[0], trans=trans, out=out)
        image = out[:size].view(torch.bfloat16).view(batch, groups, blocks, 3, 128, 32)
        for z in range(0, batch, 64):
            part = image[z:z + 64].float().sum(3)            # (24 bits in three pieces: exact in any order)
            part = part.gather(-1, at.expand(part.shape)).permute(0, 2, 3, 1, 4).reshape(part.shape[0], blocks * 128, groups * 32)
            assert torch.equal(part[:, :rows, :K], x[z:z + 64].abs()), (where, z)
            assert not part[:, :rows, K:].any() and not part[:, rows:(rows + 3) // 4 * 4].any()
        marks = out[size:size + 512]
        if K > 256:                                          # (no form reads shorter ones')
            assert bool((marks == 0xa5).all()) == (where is None) and set(marks.unique().tolist()) <= {0, 0xa5}, where
        if where:
            x[where] = 1.0
