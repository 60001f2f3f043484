"""The one-pass checks of rows, dealt out over workgroups and trips: every row counts once, whatever their number is, and nothing behind the last
one does.  The profile is that of the stored bound and the streaming check, field for field."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tao():
    import paper_2510_16028_amd as t
    t.lib()
    return t


def _same(got, want, what):
    assert set(got) == set(want)
    for key in want:
        a, b = np.asarray(got[key]), np.asarray(want[key])
        assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f"), (what, key, got[key], want[key])


# lanes of a row group and columns of its rows; a workgroup has 1024 lanes, the chip 256 workgroups
@pytest.mark.parametrize("lanes,cols", [(16, 60), (32, 100), (64, 200), (64, 512), (256, 777), (256, 1500), (512, 2052)])
def test_rows_dealt_out(tao, lanes, cols):
    groups = 1024 // lanes
    counts = {2 * groups, 2 * groups + 1, 17 * groups - 1, 255, 256, 257, 511, 256 * groups - 1, 256 * groups, 256 * groups + 1, 300 * groups + 5,
              512 * groups, 513 * groups - 1, 700 * groups + 1, 1024 * groups, 1024 * groups + 1, 1100 * groups}
    g = torch.Generator(device="cuda").manual_seed(cols)
    for rows in sorted(c for c in counts if c * cols <= 9_000_000):
        def place(t):                                        # (rows of NaN behind the last one)
            return torch.cat([t, torch.full((64, cols), float("nan"), device="cuda")])[:rows]

        x = torch.randn((rows, cols), generator=g, device="cuda")
        claims = lambda y: torch.where(torch.rand(y.shape, generator=g, device="cuda") < 0.001, y * 1.01,
                                       (y.double() * (1 + 2.0 ** -24 * torch.randint(-2, 3, y.shape, generator=g, device="cuda"))).float())
        for kind in (tao.NORM_LAYERNORM, tao.NORM_RMSNORM):
            y = x * 0.7 if kind == tao.NORM_RMSNORM else x - 0.1
            c = claims(y)
            want = tao.tao_check_and_profile(c, y, tao.tao_bound_norm(kind, x, y, None, None, eps=1e-5))
            _same(tao.tao_bound_check_norm(kind, place(x), place(y), place(c), None, None, eps=1e-5), want, (kind, rows))
        y = torch.softmax(x, dim=-1)
        c = claims(y)
        want = tao.tao_check_and_profile(c, y, tao.tao_bound_softmax(x, y))
        _same(tao.tao_bound_check_softmax(place(x), place(y), place(c)), want, ("softmax", rows))
