"""Which form of the screen checks a product, by the launch: that the shapes that are tested on the device reach the forms they are meant for, and
that operands are marked where a form reads the marks."""
import launches
from test_gpu_screen_first_slab import SHAPES

BODY = r"""
P = address(1 << 20)
SHAPES = %r
result = []
for form, shapes in SHAPES.items():
    for batch, M, N, K in shapes:
        # (prepared images, and operands that the call cuts)
        assert lib.tao_bound_check_linear_images(P, P, None, P, P, None, M, N, K, N, batch, M * N, 0, 1.0, 1e-12, None, P, P, 1 << 40, None) == 0
        result.append((form, batch, M, N, K, 1, [l[0] for l in launched()]))
        assert lib.tao_bound_check_linear(P, P, None, P, P, None, M, N, K, K, K, N, 0, batch, M * K, N * K, M * N, 1.0, 1e-12, None, P, P, 1 << 40, None) == 0
        result.append((form, batch, M, N, K, 0, [l[0] for l in launched()]))
"""


def test_every_shape_reaches_its_form(tmp_path):
    found = launches.run(BODY % SHAPES, tmp_path)
    assert len(found) == 2 * sum(len(shapes) for shapes in SHAPES.values())
    for form, batch, M, N, K, images, kernels in found:
        case = (batch, M, N, K, kernels)
        screen, cut = [k for k in kernels if k.startswith("screen_product<")], [k for k in kernels if k.startswith("split3_bf16<")]
        if images:
            assert len(screen) == 1 and screen[0].startswith("screen_product<" + form) and not cut, case
        elif screen:                                         # (or binary32 rows, and products that are not screened)
            tries = screen[0].split("<")[1].split(", ")[8]
            assert len(cut) == 1 and cut[0] == "split3_bf16<" + tries, case


CONVOLUTIONS = r"""
P = address(1 << 20)
result = []
for C, R in ((32, 1), (64, 1), (96, 1), (128, 1), (32, 3)):
    assert lib.tao_bound_check_conv2d(P, P, None, P, P, None, 32, 28, 28, C, 512, R, R, 1, 1, R // 2, R // 2, 1, 1, 1.0, 1e-12, None, P, P, 1 << 40, None) == 0
    result.append((C * R * R, [l[0] for l in launched()]))
"""


def test_a_convolution_of_one_slab_tries_none(tmp_path):
    for K, kernels in launches.run(CONVOLUTIONS, tmp_path):
        tries = "true" if K > 64 else "false"
        assert [k for k in kernels if k.startswith("split3_bf16<")] == ["split3_bf16<" + tries], (K, kernels)
        assert [k.split("<")[1].split(", ")[8] for k in kernels if k.startswith("screen_product<2, 2, 2, 2, 2, 2, 2, 2, ")] == [tries], (K, kernels)
