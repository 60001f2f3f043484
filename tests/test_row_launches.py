"""Launches of the one-pass row checks, by their arguments: of empty tensors, and how rows are dealt out."""
import launches

# the constants' last two fields
CONSTS = r"""
class Consts(ctypes.Structure):
    _fields_ = [("numbers", ctypes.c_double * 12), ("quick_alpha", ctypes.c_float), ("apart", ctypes.c_int)]
P = address(1 << 20)
def softmax(rows, cols, p=P):
    watch("softmax_check", (3, ctypes.c_long), (6, Consts))
    assert lib.tao_bound_check_softmax(p, p, p, rows, cols, cols, 1.0, 1e-12, None, P, P, 1 << 24, None) == 0
    return launched()[0]
def norm(kind, rows, cols, p=P):
    watch("norm_check", (4, ctypes.c_long), (7, Consts))
    assert lib.tao_bound_check_norm(kind, p, p, p, p, 1e-5, p, rows, cols, cols, 1.0, 1e-12, None, P, P, 1 << 24, None) == 0
    return launched()[0]
calls = {"softmax": softmax, "layernorm": lambda *a: norm(tao.NORM_LAYERNORM, *a), "rmsnorm": lambda *a: norm(tao.NORM_RMSNORM, *a)}
"""

EMPTY = CONSTS + r"""
result = []
for name, call in calls.items():
    for rows, cols in ((0, 16), (0, 5000), (7, 0), (0, 0)):
        kernel, grid, block, (r, k) = call(rows, cols, None)
        result.append((name, rows, cols, kernel, grid, block, r.value, k.apart))
"""


def test_an_empty_tensor_gives_a_kernel_no_rows(tmp_path):
    found = launches.run(EMPTY, tmp_path)
    assert len(found) == 3 * 4
    for name, rows, cols, kernel, grid, block, r, apart in found:
        case = (name, rows, cols)
        assert kernel.startswith("softmax_check<" if name == "softmax" else "norm_check<") and (grid, block) == (1, 1024), case
        assert r == 0 and apart == 1, (case, r, apart)           # row group s begins at row s, of none


DEALT = CONSTS + r"""
result = []
for name, call in calls.items():
    for rows in (1, 2, 3, 17, 255, 256, 257, 4095, 4096, 4097, 8192, 20001):
        for cols in (1, 3, 4, 61, 128, 200, 512, 513, 1024, 1500, 2048, 4096, 8200):
            kernel, grid, block, (r, k) = call(rows, cols)
            result.append((kernel, grid, block, r.value, k.apart, cols))
"""


def test_every_row_belongs_to_one_row_group(tmp_path):
    """The rows that a kernel's row groups walk, by its threads per row, grid and the distance of neighbouring ones: each row once."""
    found = launches.run(DEALT, tmp_path)
    assert len(found) == 3 * 12 * 13
    for kernel, grid, block, rows, apart, cols in found:
        inside = kernel[kernel.index("<") + 1:].split(",")
        tpr = int(inside[0] if kernel.startswith("softmax") else inside[1])
        groups, seen = block // tpr, [0] * rows
        assert apart >= 1 and 1 <= grid <= 256, (kernel, grid, rows, apart)
        for b in range(grid):
            for s in range(groups):
                for row in range(b * (groups if apart == 1 else 1) + apart * s, rows, grid * groups):
                    seen[row] += 1
        assert seen == [1] * rows, (kernel, grid, rows, apart, cols)


TRIPS = CONSTS + r"""
result = [(name, rows, cols) + call(rows, cols)[1:2] + (call(rows, cols)[3][1].apart,)
          for name, call in calls.items() for rows, cols in ((16384, 300), (8192, 2048), (16384, 1024), (9000, 300), (9000, 2048))]
"""


def test_rows_of_whole_trips_stay_together(tmp_path):
    """Neighbouring rows where every trip is a full one, but for a wavefront's rows of four vectors; otherwise the last trip is everybody's."""
    for name, rows, cols, grid, apart in launches.run(TRIPS, tmp_path):
        assert apart == (1 if rows != 9000 and cols != 1024 else grid), (name, rows, cols, grid, apart)


FORMS = CONSTS + r"""
result = [(name, rows, cols, call(rows, cols)[0]) for name, call in calls.items()
          for rows, cols in ((38, 51), (100000, 51), (38, 126), (100000, 126), (38, 130), (16384, 130), (30000, 130), (38, 195), (30000, 195), (38, 128), (38, 132))]
"""


def test_ragged_rows_of_a_wavefront_are_read_by_what_a_lane_has(tmp_path):
    """By single values where a lane has one or two, or three in few rows; by vectors otherwise."""
    for name, rows, cols, kernel in launches.run(FORMS, tmp_path):
        args = kernel.split("<")[1].split(", ")[0 if name == "softmax" else 1:]
        if args[0] != "64":                                  # (the norms' short rows: sixteen lanes, thirty-two)
            continue
        single, whole, vectors = "0", "1", "2"
        want = whole if cols % 4 == 0 else single if cols <= 128 or (cols <= 192 and rows < 24576) else vectors
        assert args[:3] == ["64", "1", want], (name, rows, cols, kernel)
