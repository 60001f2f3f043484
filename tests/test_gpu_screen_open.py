"""What the screen of a checked matmul bound leaves open, and what settles it: the records in the workspace hold the comparisons
that the one product cannot decide, by place or by block, and nothing else; the profile is the stored bound's in every case."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

LIST = 14                                                    # places that a tile's record holds


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


class Product:
    """A checked bound on a workspace of exactly the size asked for, its stored bound, and the records after a call.  form: both
    operands as images, both as matrices, or a 1 x 1 convolution (rows its pixels).  The workspace: images of the operands, sums of a reduction's
    parts, the check's partial results (64 histograms of 2048 words, then the records), a stored bound, a convolution's magnitudes."""

    def __init__(self, tao, form, batch, M, N, K, seed=0):
        self.tao, self.batch, self.M, self.N = tao, batch, M, N
        g = self.g = torch.Generator(device="cuda").manual_seed(seed + M + N + K)
        shape = (batch,) if batch > 1 else ()
        A, W = torch.randn((*shape, M, K), generator=g, device="cuda"), torch.randn((*shape, N, K), generator=g, device="cuda") * 0.1
        self.A, self.W = A, W
        self.out = tao.new_profile_buffer(A.device)
        r256 = lambda n: (int(n) + 255) // 256 * 256
        behind = r256(tao.tao_check_workspace_bytes(1)) + (r256(4 * batch * M * N) if K < 1025 else 0)
        if form == "pixels":
            assert batch == 1 and tao.tao_conv2d_split_supported((1, 1, M, K), (N, 1, 1, K))
            n = tao.lib().tao_conv2d_split_workspace_bytes(1, 1, M, K, N, 1, 1, 1, 1, 0, 0, 1, 1, 1)
            behind += M * K * 2 + 64
            self.bound = lambda: tao.tao_bound_conv2d_split(A.view(1, 1, M, K), W.view(N, 1, 1, K)).view(M, N)
            self.call = lambda y, c, ws: tao.tao_bound_check_conv2d(A.view(1, 1, M, K), W.view(N, 1, 1, K), None, y.view(1, 1, M, N), c.view(1, 1, M, N),
                                                                    out=self.out, ws=ws)
        else:
            self.bound = lambda: tao.tao_bound_linear_split(A, W)
            if form == "images":
                n = tao.lib().tao_check_linear_images_workspace_bytes(M, N, K, batch)
                self.call = lambda y, c, ws: tao.tao_bound_check_linear_images(tao.tao_split_operand(A), tao.tao_split_operand(W), M, N, K, y, c, batch=batch,
                                                                               shared_w=False, out=self.out, ws=ws)
            else:
                n = tao.tao_bound_check_linear_workspace_bytes(M, N, K, batch, batch == 1)
                self.call = lambda y, c, ws: tao.tao_bound_check_linear(A, W, None, y, c, out=self.out, ws=ws)
        self.tiles = (batch, (M + 127) // 128, (N + 127) // 128)
        self.at = int(n) - behind + 64 * 2048 * 4
        self.ws = torch.empty(int(n), dtype=torch.uint8, device="cuda")
        # (outputs of the size of their bounds, so that a claim's rounding moves it by no more than 2^-23 of the bound)
        self.tau = self.bound()
        self.y = self.tau * torch.randn(self.tau.shape, generator=g, device="cuda")

    def check(self, c):
        """Compares the profile with the stored bound's; (blocks, places) of every record."""
        want = self.tao.tao_check_and_profile(c, self.y, self.tau)
        _same(self.call(self.y, c, self.ws), want)
        n = int(np.prod(self.tiles))
        rec = self.ws[self.at:self.at + n * 64].cpu().numpy().view(np.uint32).reshape(*self.tiles, 16)
        return rec[..., 0] & 0xffff, rec[..., 0] >> 16, rec

    def honest(self):
        pick = torch.randint(-2, 3, self.y.shape, generator=self.g, device="cuda")
        return (self.y.double() * (1 + 2.0 ** -23 * pick)).float()

    def at_bound(self, f=1.0):
        return (self.y.double() + f * self.tau.double()).float()


# launch configurations of the screen, with and without a reduction in parts
FORMS = [("images", 1, 2050, 2052, 288), ("images", 1, 2050, 2052, 96), ("images", 1, 1000, 1500, 96), ("images", 1, 300, 200, 2080), ("images", 3, 200, 270, 64),
         ("matrices", 1, 300, 200, 1056), ("matrices", 12, 512, 64, 512), ("matrices", 1, 33000, 100, 1056), ("matrices", 1, 301, 1003, 333),
         ("pixels", 1, 33000, 256, 128), ("pixels", 1, 20000, 96, 64)]


@pytest.mark.parametrize("form,batch,M,N,K", FORMS)
def test_what_is_left_open(tao, form, batch, M, N, K):
    p = Product(tao, form, batch, M, N, K)
    nothing = lambda c: not p.check(c)[2].any()
    honest = p.honest()
    assert nothing(honest) and nothing(p.y.clone())
    f = torch.tensor([0.5, 0.985, 1.015, -1.015, 3.0], dtype=torch.float64, device="cuda")
    assert nothing((p.y.double() + f[torch.randint(0, 5, p.y.shape, generator=p.g, device="cuda")] * p.tau.double()).float())
    c = honest.clone()
    c.view(-1)[::7] = float("nan"); c.view(-1)[3::7] = float("inf"); c.view(-1)[5::7] = -3e38
    assert nothing(c)                                        # (violations of every bound)
    # one place in the last tile: at the bound, and near enough for the product but not for the real sum
    for f in (1.0, 1 + 1e-4, 1 - 1e-4, 1.003, 0.997):
        c = honest.clone()
        c.view(-1)[-1] = p.at_bound(f).view(-1)[-1]
        blocks, places, rec = p.check(c)
        assert not blocks.any() and places.sum() == 1 and places[-1, -1, -1] == 1
        assert rec[-1, -1, -1, 2] == ((M - 1) % 128) * 128 + (N - 1) % 128
    # as many places of one block as a record holds, and one more
    near = p.at_bound()
    for n in (LIST, LIST + 1):
        c = honest.clone()
        pick = torch.randperm(32 * 32, generator=p.g, device="cuda")[:n]
        z = (batch - 1,) if batch > 1 else ()
        c[(*z, pick // 32, pick % 32)] = near[(*z, pick // 32, pick % 32)]
        blocks, places, rec = p.check(c)
        if n <= LIST:
            assert not blocks.any() and places.sum() == n
            assert sorted(rec[-1, 0, 0, 2:2 + n]) == sorted((pick // 32 * 128 + pick % 32).tolist())
        else:
            assert blocks[-1, 0, 0] & 1 and (blocks != 0).sum() == 1 and not places.any()
    # two blocks that ask for more places than there are: one of them is taken whole
    c = honest.clone()
    z = (0,) if batch > 1 else ()
    c[(*z, 3, slice(0, 8))], c[(*z, 70, slice(8, 16))] = near[(*z, 3, slice(0, 8))], near[(*z, 70, slice(8, 16))]
    blocks, places, rec = p.check(c)
    assert places.sum() == 16 and (blocks != 0).sum() == 1 and blocks[0, 0, 0] in (1, 3, 0x11, 0x33, 0x100, 0x300, 0x1100, 0x3300)
    # all of it
    blocks, places, _ = p.check(p.at_bound())
    assert ((blocks != 0) | (places != 0)).all()             # (a corner of few elements is a list)


@pytest.mark.parametrize("form,batch,M,N,K", FORMS)
def test_an_operand_that_is_not_screened_opens_its_tiles(tao, form, batch, M, N, K):
    p = Product(tao, form, batch, M, N, K, seed=1)
    for value in (2.0 ** 32, float("inf"), float("nan")):
        p.A.view(-1)[-K // 2] = value                        # the last row, of the last batch entry
        p.tau = p.bound()
        c = p.honest()
        blocks, places, _ = p.check(c)
        assert (blocks[-1, -1] != 0).all() and not places.any()
        assert not blocks[:-1].any() and not blocks[-1, 0].any()


# several tiles to a workgroup of each configuration: after one that is open everywhere no further products are formed
@pytest.mark.parametrize("form,batch,M,N,K", [("images", 1, 3000, 3100, 288), ("images", 1, 4200, 2200, 64), ("images", 1, 70000, 64, 96),
                                              ("matrices", 1, 66000, 100, 64), ("matrices", 1, 40000, 64, 96), ("pixels", 1, 70000, 64, 32),
                                              ("pixels", 1, 70000, 130, 64)])
def test_open_regions(tao, form, batch, M, N, K):
    p = Product(tao, form, batch, M, N, K)
    near = (p.y.double() + (1 + 2e-3 * torch.randn(p.y.shape, generator=p.g, device="cuda", dtype=torch.float64)) * p.tau.double()).float()
    rows, cols = torch.arange(M, device="cuda")[:, None], torch.arange(N, device="cuda")[None, :]
    for where in (rows >= 0, rows < M // 3, cols >= N // 2, (rows // 128 + cols // 128) % 5 == 0, (rows % 128 < 30) & (cols % 128 < 30), torch.rand((M, N), generator=p.g, device="cuda") < 0.01):
        p.check(torch.where(where, near, p.honest()))


@pytest.mark.parametrize("M,N", [(2, 3), (8, 4)])
def test_more_tiles_than_whole_records(tao, M, N):
    """25000 batch entries are as many tiles: their records lie where the bound of so short a reduction would be stored, or, where that is
    too small for them, are the state alone, without places."""
    B, K = 25000, 40
    g = torch.Generator(device="cuda").manual_seed(2)
    A, W = torch.randn((B, M, K), generator=g, device="cuda"), torch.randn((B, N, K), generator=g, device="cuda")
    tau = tao.tao_bound_linear_split(A, W)
    y = tau * torch.randn(tau.shape, generator=g, device="cuda")
    honest = y * (1 + 2.0 ** -23)
    for share in (0.0, 1e-4, 0.3, 1.0):
        near = (y.double() + (1 + 2e-3 * torch.randn(y.shape, generator=g, device="cuda", dtype=torch.float64)) * tau.double()).float()
        c = torch.where(torch.rand(y.shape, generator=g, device="cuda") < share, near, honest)
        _same(tao.tao_bound_check_linear(A, W, None, y, c), tao.tao_check_and_profile(c, y, tau))
