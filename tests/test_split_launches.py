"""How an operand is dealt out to the workgroups that cut it, by the launch: each leaves a mark where a product can read them, of which there are 512, and few of them
leave the chip idle."""
import launches

CUT = r"""
result = []
P = address(1 << 20)
for rows, K, trans, batch in ((64, 32, 0, 1), (64, 512 * 32, 0, 1), (64, 513 * 32, 0, 1), (739, 739, 0, 2), (600, 1700, 1, 1), (1500, 1500, 0, 1), (3072, 768, 0, 1),
                              (1111, 1001, 0, 1), (4096, 1024, 0, 1), (4096, 1056, 0, 1), (12288, 4096, 0, 1), (8, 4 * 513 * 32, 0, 1), (64, 64, 0, 3000), (64, 256, 0, 300), (64, 257, 0, 300)):
    assert lib.tao_split_operand(P, rows, K, rows if trans else K, trans, batch, rows * K, P, 1 << 40, None) == 0
    (kernel, grid, block, _), = launched()
    units = (K + 31) // 32 * ((rows + 63) // 64) * batch
    result.append((kernel, rows, K, batch, units, grid, block))
"""


def test_an_operand_is_cut_on_all_of_the_chip(tmp_path):
    found = launches.run(CUT, tmp_path)
    assert len(found) == 15
    for kernel, rows, K, batch, units, grid, block in found:
        case = (rows, K, batch, units, grid, block)
        assert kernel == "split3_bf16<" + ("true" if K > 256 else "false"), case
        if K <= 256:                                         # (read by products without first slabs only)
            assert (grid, block) == (units, 256), case
            continue
        assert 1 <= grid <= 512 and block in (256, 512, 768, 1024), case
        if rows <= 16:                                       # (a wavefront to a unit)
            units = (units + 3) // 4
        assert grid == min(units, 512), case                 # two workgroups to a compute unit as soon as there are units for them
        assert block // 256 == min(4, -(-units // 512)), case        # and no more threads in each than units ask for


BOTH = r"""
result = []
P = address(1 << 20)
for M, N, K in ((1892, 576, 2560), (1500, 1000, 1000), (1500, 700, 1500), (576, 1892, 2560), (1400, 1300, 500), (1000, 300, 400)):
    assert lib.tao_bound_check_linear(P, P, None, P, P, None, M, N, K, K, K, N, 0, 1, 0, 0, 0, 1.0, 1e-12, None, P, P, 1 << 40, None) == 0
    result.append((M, N, K, [l[:3] for l in launched() if l[0] == "split3_bf16<true"]))
"""


def test_the_shorter_of_two_operands_fills_its_workgroups(tmp_path):
    found = launches.run(BOTH, tmp_path)
    assert len(found) == 6
    for M, N, K, cuts in found:
        (_, grid, block), = cuts
        units = sorted(-(-K // 32) * -(-rows // 64) for rows in (M, N))
        parts = min(4, -(-units[1] // 512))
        shorter = units[0] if -(-units[0] // 512) == parts else -(-units[0] // parts)
        assert (grid, block) == (min(units[1], 512) + min(shorter, 512), 256 * parts), (M, N, K, units, grid, block)


READERS = r"""
result = []
P = address(1 << 20)
for K in (1, 64, 128, 256, 257, 288, 384, 385, 512, 4096):
    for batch, M, N in ((1, 64, 64), (1, 300, 300), (1, 2048, 1024), (1, 2048, 64), (1, 4096, 4096), (8, 2048, 2048)):
        assert lib.tao_bound_check_linear_images(P, P, None, P, P, None, M, N, K, N, batch, M * N, 0, 1.0, 1e-12, None, P, P, 1 << 40, None) == 0
        result.append((batch, M, N, K, [l[0] for l in launched() if l[0].startswith("screen_product<")]))
"""


def test_a_product_reads_no_marks_that_its_operands_do_not_have(tmp_path):
    tries = set()
    for batch, M, N, K, screen in launches.run(READERS, tmp_path):
        if screen and screen[0].split("<")[1].split(", ")[8] == "true":
            assert K > 256, (batch, M, N, K, screen)
            tries.add(K)
    assert {288, 385} <= tries
