"""The FP32 tiles of the matmul bound at output sizes that are left to them (small outputs run on the binary64 matrix
cores): ragged and unaligned operands, all modes, subnormal sums, and launches of both tile heights; sampled rows
against the oracle."""
import numpy as np
import pytest
import torch

from opmap import assert_bound_parity

pytestmark = pytest.mark.gpu

# The binary64 route stays within one binary32 step (2^-23) of the oracle; the FP32 scheme's inflation alone is 7 x 2^-24.
ONE_STEP = 1.3e-7


@pytest.fixture(scope="module")
def tao():
    import paper_2510_16028_amd as t
    t.lib()
    assert torch.cuda.is_available()
    return t


def _rows(M, rng):
    """Both ends, both sides of the tiles' edges, and some more."""
    edges = [r for r in (0, 1, 31, 32, 63, 64, 127, 128, M - 65, M - 33, M - 2, M - 1) if 0 <= r < M]
    return np.unique(np.concatenate([edges, rng.integers(0, M, 20)]))


def _operands(rng, M, N, K, trans_w, batch, ld_pad, offset, scale=(1.0, 1.0)):
    """A [batch][M][K] and W as views with `ld_pad` further columns, starting `offset` floats into a row."""
    def view(rows, cols, s):
        wide = torch.from_numpy(rng.standard_normal((batch, rows, cols + ld_pad)).astype(np.float32)) * s
        return wide.cuda()[:, :, offset:offset + cols]
    A, W = view(M, K, scale[0]), view(K if trans_w else N, N if trans_w else K, scale[1])
    return (A[0], W[0]) if batch == 1 else (A, W)


def _compare(oracle_mod, got, A, W, bias, trans_w, rng, model=None):
    """Pairs (bound, oracle's) on sampled rows of every batch entry, as arrays."""
    rows = _rows(A.shape[-2], rng)
    g, o = [], []
    for z in range(A.shape[0] if A.dim() == 3 else 1):
        a, w, t = (A[z], W[z], got[z]) if A.dim() == 3 else (A, W, got)
        g.append(t[torch.from_numpy(rows).cuda()].cpu().numpy())
        o.append(oracle_mod.bound_linear(a[torch.from_numpy(rows).cuda()].cpu().numpy(), w.cpu().numpy(), bias, trans_w=trans_w,
                                         **({} if model is None else dict(model=model))))
    return np.concatenate(g), np.concatenate(o)


@pytest.mark.parametrize("M,N,K,bias,trans_w,batch,ld_pad,offset", [
    (2100, 1100, 199, False, False, 1, 4, 1),          # rows misaligned by 4 bytes, a ragged last group, ragged tiles
    (2100, 1100, 199, True, True, 1, 3, 2),
    (1111, 3001, 37, True, False, 1, 0, 0), (1400, 1700, 100, False, True, 1, 5, 0),
    (1300, 2200, 21, True, False, 1, 1, 1), (2000, 1900, 115, False, False, 1, 4, 4),
    (700, 650, 60, True, True, 5, 2, 1),               # batched
    (384, 384, 224, True, False, 12, 0, 0),            # aligned 64-row tiles, odd number of groups, batched
    (2048, 2048, 1056, False, False, 1, 0, 0),         # aligned 128-row tiles, just past the persistent limit
    (2100, 2100, 1031, True, False, 1, 0, 0),          # a long ragged reduction
])
def test_fp32_tiles(tao, oracle_mod, M, N, K, bias, trans_w, batch, ld_pad, offset):
    rng = np.random.Generator(np.random.Philox(M + 3 * N + K))
    A, W = _operands(rng, M, N, K, trans_w, batch, ld_pad, offset)
    b = rng.standard_normal(N).astype(np.float32) if bias else None
    bg = None if b is None else torch.from_numpy(b).cuda()
    what = str((M, N, K, bias, trans_w, batch, ld_pad, offset))
    g, o = _compare(oracle_mod, tao.tao_bound_linear(A, W, bg, trans_w=trans_w), A, W, b, trans_w, rng)
    assert assert_bound_parity(g, o, what) > ONE_STEP, "not on the FP32 tiles: " + what
    # the probabilistic constant (lambda = 4)
    got = tao.tao_bound_linear(A, W, bg, trans_w=trans_w, model=tao.FpModel(mode=1))
    g, o = _compare(oracle_mod, got, A, W, b, trans_w, rng, model=oracle_mod.Model(mode=1))
    assert_bound_parity(g, o, what + " probabilistic")
    # one chain over the reduction: looser by at most about 2 K u
    got = tao.tao_bound_linear(A, W, bg, trans_w=trans_w, model=tao.FpModel(flags=tao.FLAG_FAST_ACCUM))
    g, o = _compare(oracle_mod, got, A, W, b, trans_w, rng)
    assert_bound_parity(g, o, what + " fast", rel_tol=2.5 * K * 2.0 ** -24)


@pytest.mark.parametrize("sa,sw", [(1e-30, 1e-12), (1e-20, 1e-20), (1e-25, 1e-12), (1e-38, 1.0), (1e-19, 1e-19)])
@pytest.mark.parametrize("M,N,K,ld_pad", [(1300, 1500, 200, 0), (1300, 1500, 199, 3), (2048, 2048, 64, 0), (2100, 2100, 1031, 0)])
def test_fp32_tiles_on_tiny_operands(tao, oracle_mod, M, N, K, ld_pad, sa, sw):
    """Products and sums in the binary32 subnormal range or below it: never below the reference, above it by the
    absolute term Gamma(K) (1.25 K + 40) 2^-150 at most."""
    rng = np.random.Generator(np.random.Philox(M + K))
    A, W = _operands(rng, M, N, K, False, 1, ld_pad, 0, (sa, sw))
    g, o = _compare(oracle_mod, tao.tao_bound_linear(A, W), A, W, None, False, rng)
    assert (g >= o).all(), "%d elements below the reference" % int((g < o).sum())
    slack = (K * 2.0 ** -24 / (1 - K * 2.0 ** -24)) * (1.25 * K + 40) * 2.0 ** -150 * 1.01
    assert (g <= o.astype(np.float64) * (1 + 1e-6) + slack + 2.0 ** -149).all()
    # with the underflow terms: the reference's value or the next binary32 value above it
    flags = dict(flags=tao.FLAG_UNDERFLOW_TERMS)
    g, o = _compare(oracle_mod, tao.tao_bound_linear(A, W, model=tao.FpModel(**flags)), A, W, None, False, rng, model=oracle_mod.Model(flags=1))
    assert (g >= o).all() and (g <= np.nextafter(o * np.float32(1 + 1e-6), np.float32(np.inf))).all()


def test_fp32_tiles_on_vanishing_products(tao, oracle_mod):
    """Every product below 2^-150: the underflow terms alone carry the bound."""
    rng = np.random.Generator(np.random.Philox(7))
    A, W = _operands(rng, 1300, 1500, 200, False, 1, 0, 0, (1e-30, 1e-20))
    got = tao.tao_bound_linear(A, W, model=tao.FpModel(flags=tao.FLAG_UNDERFLOW_TERMS))
    g, o = _compare(oracle_mod, got, A, W, None, False, rng, model=oracle_mod.Model(flags=1))
    assert (g >= o).all() and (g <= o + np.float32(2.0 ** -149)).all()


@pytest.mark.parametrize("M,N,K,exact", [(1300, 1500, 200, False), (2048, 2048, 64, False), (40, 60, 200, True)])
def test_finite_operands_whose_products_overflow(tao, oracle_mod, M, N, K, exact):
    """Products beyond 2^128 in some rows and columns: +inf on the FP32 tiles, the bound itself on the binary64 route; never NaN,
    never below the reference, and the other elements as always."""
    rng = np.random.Generator(np.random.Philox(11))
    A, W = _operands(rng, M, N, K, False, 1, 0, 0)
    A[::3, 5::32] = 1.998 * 2.0 ** 70
    W[::2, 5::32] = -2.0 ** 66
    g, o = _compare(oracle_mod, tao.tao_bound_linear(A, W), A, W, None, False, rng)
    assert not np.isnan(g).any() and (g >= o).all()
    fits = np.isfinite(g) if not exact else np.isfinite(o)
    assert (g[fits] <= o[fits].astype(np.float64) * (1 + 1e-6)).all()
    assert np.isfinite(g[:, 1::2]).all()                     # (columns without the large operand)
