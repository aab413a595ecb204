"""K-slice counts between the powers of two: taken where a power of two leaves much of the chip idle, and summed like any other."""
import numpy as np
import pytest

import gemm_inputs as gi
import paper_2003_06324_amd as g


def test_slices_fill_the_chip():
    g.force_config(None)
    g.cost_model_scale(-1)
    # 40, 42 and 24 tiles of 128x128 or twice as many of half the size: powers of two would fill 160, 168 and 192 of 256 CUs
    for M, N, K in ((600, 912, 16608), (786, 669, 8937 // 64 * 64), (744, 488, 48576)):
        tile, slices = g.query_config(2, M, N, K, 16, g.ROW_MAJOR, g.COL_MAJOR).split(":s")
        bm, bn = (int(x) for x in tile[1:].split("x"))
        assert -(-M // bm) * -(-N // bn) * int(slices) > 200, (M, N, K, tile, slices)


@pytest.mark.gpu
@pytest.mark.parametrize("slices", [3, 5, 7, 10, 14, 28])
def test_exact_on_whole_numbers(oracle, slices):
    from gpu_util import run_gpu
    for dtype, tile, K in (("f16", "t128x128", 64 * 2 * slices + 40), ("bf16", "t64x128", 64 * slices), ("f32", "t64x64", 32 * slices + 7)):
        M, N = 200, 264
        A, B = gi.make_problem(70 + slices, M, N, K, "int", dtype)
        bits = (gi.bfloat16_bits(A), gi.bfloat16_bits(B)) if dtype == "bf16" else (A, B)
        ref = oracle.gemm(M, N, K, bits[0], 0, bits[1], 0, dtype)
        for la, lb in ((0, 0), (1, 1)):
            C = run_gpu(dtype, A, B, la, lb, force="%s:s%d" % (tile, slices))
            assert np.array_equal(C.astype(np.float64), ref), (dtype, la, lb)
