"""Which kernel forms a convolution's stored bound, by the launch, at shapes that were measured on both: the binary64 matrix cores or the FP32 tiles, these
also with one accumulation chain."""
import launches

# (batch, height = width, channels, filters, filter size, stride): us on binary64, on FP32 tiles, on FP32 tiles with TAO_FLAG_FAST_ACCUM
MEASURED = {
    (1, 7, 512, 64, 3, 1): (18.4, 605.0, 518.0), (4, 12, 512, 64, 3, 1): (18.8, 377.0, 328.0), (5, 31, 512, 256, 3, 1): (259.0, 360.0, 318.0),
    (3, 18, 128, 512, 3, 1): (27.2, 87.0, 74.8), (1, 56, 64, 64, 3, 1): (12.4, 51.2, 45.0), (8, 35, 100, 128, 3, 1): (70.2, 82.0, 72.3),
    (2, 28, 256, 512, 3, 2): (31.8, 171.0, 150.0), (1, 40, 256, 128, 3, 1): (31.9, 110.0, 80.9), (5, 23, 64, 512, 3, 1): (50.0, 47.0, None),
    (16, 32, 32, 512, 3, 1): (181.0, 65.0, None), (3, 33, 32, 256, 3, 1): (24.4, 24.5, 21.2), (3, 40, 128, 128, 3, 1): (46.1, 57.9, 43.7),
    (4, 28, 256, 256, 3, 1): (92.5, 110.5, 81.9), (1, 24, 128, 512, 3, 1): (27.3, 57.6, 43.2), (3, 32, 64, 128, 3, 1): (17.9, 31.4, 24.2),
    (5, 24, 512, 256, 3, 1): (156.0, 216.0, 158.0),
}

BODY = r"""
P = address(1 << 20)
result = []
for b, h, c, co, f, st in %r:
    for fast in (0, 1):
        model = tao.tao_default_model()
        model.flags |= tao.FLAG_FAST_ACCUM * fast
        assert lib.tao_bound_conv2d(P, P, None, P, b, h, h, c, co, f, f, st, st, f // 2, f // 2, 1, 1, ctypes.byref(model), None) == 0
        (kernel, _, _, _), = launched()
        result.append(((b, h, c, co, f, st), fast, kernel))
"""


def test_the_faster_kernel_is_launched(tmp_path):
    found = launches.run(BODY % list(MEASURED), tmp_path)
    assert len(found) == 2 * len(MEASURED)
    for shape, fast, kernel in found:
        f64, exact, chain = MEASURED[tuple(shape)]
        tiles = chain if fast else exact
        if tiles is None:
            continue
        here = kernel.startswith("absgemm_f64<")
        # (the rule leans to the tiles, which convolutions had before: never the slower kernel on binary64, and little of its gain left out)
        if here:
            assert f64 <= 1.04 * tiles, (shape, fast, kernel)
        else:
            assert tiles <= 1.25 * f64, (shape, fast, kernel)
