"""The one-pass checks of rows whose length fits no vector, at any alignment, and of rows that a part of a wavefront holds: the profile is that of
the stored bound and the streaming check, field for field, on both sides of the rules between the forms."""
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


# row groups of 16, 32, 64 ... 1024 lanes, one to four vectors each; by vectors and by single values (four fifths of 512, 2048, 4096 and 8192)
COLS = [1, 2, 3, 4, 5, 7, 15, 16, 17, 61, 63, 64, 65, 66, 127, 128, 129, 131, 191, 193, 255, 257, 259, 409, 410, 511, 513, 767, 1023, 1025, 1639, 2047, 2049, 3277, 4095, 5211, 6555, 8191, 8193]


def _claims(y, tau, g):
    pick = torch.randint(-2, 3, y.shape, generator=g, device="cuda")
    honest = (y.double() * (1 + 2.0 ** -24 * pick)).float()
    mixed = honest.clone()
    u = torch.rand(y.shape, generator=g, device="cuda")
    mixed = torch.where(u < 0.01, (y.double() + 3 * tau.double()).float() + 1e-30, mixed)
    mixed = torch.where(u > 0.995, float("nan"), mixed)
    mixed[-1, -1] = y[-1, -1] * 2 + 1                        # (the last element of all)
    return dict(equal=y.clone(), honest=honest, mixed=mixed)


@pytest.mark.parametrize("cols", COLS)
def test_rows(tao, cols):
    g = torch.Generator(device="cuda").manual_seed(cols)
    for rows in (1, 3, 67, 20000 if cols <= 600 else 2100) + ((26000,) if 128 < cols < 200 else ()):
        if rows * cols > 12_000_000:
            continue
        for pad, shift in ((0, 0), (3, 0), (4 - cols % 4 if cols % 4 else 0, 0), (0, 1)):
            if (pad or shift) and rows not in (67, 20000, 26000):
                continue
            ld = cols + pad

            def place(t):                                    # (what lies between and behind the rows must not count)
                flat = torch.full((rows * ld + 8,), float("nan"), device="cuda")
                view = flat[shift:shift + rows * ld].view(rows, ld)[:, :cols]
                view.copy_(t)
                return view

            x = torch.randn((rows, cols), generator=g, device="cuda") + 0.1
            gamma = 1 + 0.1 * torch.randn(cols, generator=g, device="cuda")
            for kind in (tao.NORM_LAYERNORM, tao.NORM_RMSNORM):
                y = x * 0.7 if kind == tao.NORM_RMSNORM else x - 0.1
                eps = 1e-5
                tau = tao.tao_bound_norm(kind, x, y, gamma, None, eps=eps)
                for name, c in _claims(y, tau, g).items():
                    for eps_rel in (1e-12, 0.0) if rows == 67 else (1e-12,):
                        want = tao.tao_check_and_profile(c, y, tau, eps_rel=eps_rel)
                        got = tao.tao_bound_check_norm(kind, place(x), place(y), place(c), gamma, None, eps=eps, eps_rel=eps_rel)
                        _same(got, want, (kind, rows, pad, shift, name, eps_rel))
            if cols > 1:
                xm = x.clone()
                xm[rows // 2, cols // 2:] = float("-inf")
                y = torch.softmax(xm, dim=-1)
                tau = tao.tao_bound_softmax(xm, y)
                for name, c in _claims(y, tau, g).items():
                    _same(tao.tao_bound_check_softmax(place(xm), place(y), place(c)), tao.tao_check_and_profile(c, y, tau), ("softmax", rows, pad, shift, name))
