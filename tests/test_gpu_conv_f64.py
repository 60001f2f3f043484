"""The convolution bound of few output pixels, on the binary64 matrix cores: tau against the sum of magnitudes in 64 bits, one-sided
within 1e-6, at the edges of the tiles, of the reduction's chunks and of the image, on both sides of the rule that chooses the kernel."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


# (batch, height, width, C, Cout, R, S, stride, padding, dilation, bias): channels in fours and not, one chunk of 32 k and fewer, many; a row tile's
# and a column tile's remainder; taps in the padding, a padding wider than the filter; a filter as large as the image
@pytest.mark.parametrize("B,H,W,C,Co,R,S,st,pad,dil,bias", [
    (1, 1, 1, 1, 1, 1, 1, 1, 0, 1, False), (1, 7, 7, 3, 16, 3, 3, 1, 1, 1, True), (2, 5, 9, 4, 17, 3, 1, 1, 1, 1, False), (1, 7, 7, 8, 15, 2, 2, 1, 0, 1, True),
    (3, 7, 8, 100, 33, 3, 3, 2, 1, 1, True), (1, 9, 9, 512, 64, 3, 3, 1, 1, 1, False), (5, 7, 7, 512, 65, 3, 3, 2, 1, 1, True), (2, 14, 13, 36, 100, 3, 3, 1, 2, 2, True),
    (1, 6, 6, 30, 70, 6, 6, 1, 0, 1, False), (1, 12, 12, 5, 40, 5, 3, 3, 4, 1, True), (11, 16, 16, 3, 96, 7, 7, 2, 3, 1, False), (4, 19, 19, 128, 130, 3, 3, 1, 1, 1, True),
    (13, 15, 15, 64, 512, 1, 1, 2, 0, 1, False), (9, 30, 30, 32, 256, 3, 3, 1, 1, 1, True), (20, 40, 40, 3, 64, 3, 3, 1, 1, 1, True)])
def test_bound(B, H, W, C, Co, R, S, st, pad, dil, bias):
    import paper_2510_16028_amd as tao
    g = torch.Generator(device="cuda").manual_seed(B + H * C + Co)
    # (what lies beside the image holds values that a tap outside it must not bring in)
    room = torch.full((B * H * W * C + 64,), 1e30, device="cuda")
    x = room[32:32 + B * H * W * C].view(B, H, W, C)
    x.copy_(torch.randn((B, H, W, C), generator=g, device="cuda"))
    w = torch.randn((Co, R, S, C), generator=g, device="cuda")
    b = torch.randn(Co, generator=g, device="cuda") if bias else None
    ref = torch.nn.functional.conv2d(x.double().abs().permute(0, 3, 1, 2), w.double().abs().permute(0, 3, 1, 2), None, st, pad, dil).permute(0, 2, 3, 1)
    K = R * S * C + (1 if bias else 0)
    want = (ref + (b.double().abs() if bias else 0.0)) * oracle.gamma(K)
    for shift in (0, 1):                                     # 16-byte aligned and not
        xs = room[32 - shift:32 - shift + x.numel()].view(x.shape)
        if shift:
            xs.copy_(x.clone())
        tau = tao.tao_bound_conv2d(xs, w, b, st, pad, dil).double()
        assert tau.shape == want.shape
        # (the reference's own sums of non-negative terms in 64 bits: K 2^-53 of them)
        slack = K * 2.0 ** -52
        assert bool((tau >= want * (1 - slack)).all()) and bool((tau <= want * (1 + 1e-6 + slack)).all()), (shift, float((tau / want).min()) - 1, float((tau / want).max()) - 1)


def test_infinite_operands_reach_their_outputs_only():
    import paper_2510_16028_amd as tao
    x, w = torch.ones((1, 9, 9, 64), device="cuda"), torch.ones((32, 3, 3, 64), device="cuda")
    for value in (float("inf"), float("nan"), 3e38):
        x2 = x.clone()
        x2[0, 4, 4, 63] = value
        tau = tao.tao_bound_conv2d(x2, w, None, 1, 1).cpu().numpy()[0, :, :, 0]
        near = np.zeros((9, 9), dtype=bool)
        near[3:6, 3:6] = True
        assert np.isfinite(tau[~near]).all() and (np.isnan(tau[near]).all() if value != value else (tau[near] >= min(value, 1e33)).all())
