"""The matmul bound on the binary64 matrix cores (outputs too small for the FP32 tiles): every element
against the oracle at the edges of its tiles, chunks and wavefronts, and the FP32 tiles at ragged sizes
on the other side of the rule."""
import pytest
import torch

from opmap import assert_bound_parity

pytestmark = pytest.mark.gpu

# Both sides round up to binary32 a value that is exact to (K + 64) 2^-52: at most one binary32 step apart.
ONE_STEP = 1.2e-7          # > 2^-23 (1 + 2^-20)


@pytest.fixture(scope="module")
def tao():
    import paper_2510_16028_amd as t
    t.lib()
    assert torch.cuda.is_available()
    return t


@pytest.mark.parametrize("M,N,K,bias,trans_w,batch,pad,tol", [
    (1, 1, 1, False, False, 1, 0, ONE_STEP),
    (8, 200, 1000, True, False, 1, 0, ONE_STEP),       # 16 x 16 tile, 32 chunks for 16 wavefronts, the last one ragged
    (8, 200, 1056, True, True, 1, 0, ONE_STEP),        # odd number of chunks per wavefront, W stored K x N
    (16, 17, 31, False, True, 1, 0, ONE_STEP),         # less than one chunk
    (3, 8200, 70, True, True, 1, 0, ONE_STEP),         # 16 x 32 tiles, ragged columns
    (5, 16400, 40, False, False, 1, 4, ONE_STEP),      # 16 x 64 tiles, padded rows
    (5, 16400, 608, True, True, 1, 4, ONE_STEP),       # more than one chunk per wavefront
    (20, 4100, 100, True, False, 1, 3, ONE_STEP),      # 32 x 16 tiles, unaligned rows
    (20, 8200, 300, False, True, 1, 0, ONE_STEP),      # 32 x 32 tiles
    (64, 4100, 130, True, False, 1, 0, ONE_STEP),      # 64 x 16 tiles
    (128, 4096, 601, True, False, 1, 0, ONE_STEP),     # 64 x 32 tiles: the wavefronts' sums meet in two steps
    (100, 4090, 130, False, True, 1, 0, ONE_STEP),     # the same with fewer chunks than wavefronts
    (70, 130, 513, True, False, 5, 0, ONE_STEP),       # batched
    (3001, 1111, 37, True, False, 1, 0, 1e-6), (3001, 1111, 37, False, True, 1, 0, 1e-6),      # FP32 tiles
])
def test_small_output_products(tao, oracle_mod, M, N, K, bias, trans_w, batch, pad, tol):
    g = torch.Generator().manual_seed(M * 1000 + N * 10 + K)
    A = torch.randn((batch, M, K), generator=g)
    W = torch.randn((batch, K, N) if trans_w else (batch, N, K), generator=g)
    A[:, :, K // 2] = 0.0
    A[:, M // 2] *= 1e-30                                # sums far down, still normal
    b = torch.randn((N,), generator=g) if bias else None

    def padded(t):                                       # the same values with a leading dimension beyond the row
        wide = torch.full(t.shape[:-1] + (t.shape[-1] + pad,), float("nan"))
        wide[..., :t.shape[-1]] = t
        return wide.cuda()[..., :t.shape[-1]]

    want = oracle_mod.bound_linear(A.squeeze(0).numpy() if batch == 1 else A.numpy(), W.squeeze(0).numpy() if batch == 1 else W.numpy(),
                                   None if b is None else b.numpy(), trans_w=trans_w)
    got = tao.tao_bound_linear(padded(A[0] if batch == 1 else A), padded(W[0] if batch == 1 else W), None if b is None else b.cuda(),
                               trans_w=trans_w)
    assert_bound_parity(got.cpu().numpy(), want, str((M, N, K, bias, trans_w, batch, pad)), rel_tol=tol)


# Workgroups are dealt round-robin to the XCDs: outputs of few column tiles with many row tiles or batch entries keep all
# of them busy only if the tiles, not the columns, are dealt out.  Swapping the operands transposes such an output
# into a wide one with the same bytes and products (with the columns dealt out it took 3.5 - 7 times as long).
@pytest.mark.parametrize("M,N,K,batch", [(65536, 16, 256, 1), (50176, 64, 147, 1), (512, 64, 512, 64), (8192, 16, 1024, 8)])
def test_narrow_outputs_use_the_whole_chip(tao, M, N, K, batch):
    A, W = torch.randn((batch, M, K), device="cuda"), torch.randn((batch, N, K), device="cuda")

    def us(a, w):
        out = tao.tao_bound_linear(a, w)
        times = []
        for _ in range(5):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(20):
                tao.tao_bound_linear(a, w, out=out)
            end.record()
            end.synchronize()
            times.append(start.elapsed_time(end) * 50)
        return min(times)

    narrow, wide = us(A, W), us(W, A)
    print("%d x %d x %d, batch %d: %.1f us, transposed %.1f us" % (M, N, K, batch, narrow, wide))
    assert narrow < 2 * wide
