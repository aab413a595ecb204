"""gemm_stage_kernel on K-contiguous rows that begin off the cache lines: every place of a row in its line, one or both operands,
the fewest slabs, remainders of K, ragged tiles, K-slices; and on fewer rows than the straightening needs."""
import numpy as np
import pytest

import gemm_inputs as gi
import paper_2003_06324_amd as g
from gpu_util import run_gpu

pytestmark = pytest.mark.gpu

TILES = {"t64x64": (64, 64, 32), "t64x128": (64, 128, 24), "t128x64": (128, 64, 24), "t128x128": (128, 128, 24)}


@pytest.mark.parametrize("tile", sorted(TILES))
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_exact_on_whole_numbers(oracle, tile, dtype):
    bm, bn, fewest = TILES[tile]
    for n, rem in enumerate((64, 8, 9, 63, 64, 33, 16)):
        slices = 1 + n % 2
        K = 64 * (fewest + n) * slices - 64 + rem
        M, N = ((2 * bm, 9 * bn), (bm + 1, 5 * bn - 3), (1000, 320), (7, 600))[n % 4]
        A, B = gi.make_problem(2300 + K, M, N, K, "int", dtype)
        bits = (gi.bfloat16_bits(A), gi.bfloat16_bits(B)) if dtype == "bf16" else (A, B)
        ref = oracle.gemm(M, N, K, bits[0], 0, bits[1], 0, dtype)
        for la, lb in ((0, 0), (0, 1), (1, 1)):
            # (leading dimensions of 8 (1 + n) elements past whole lines where K is contiguous, whole granules elsewhere; padding is NaN)
            pad = -K % 64 + 8 * (1 + n)
            pads = (pad if la == 0 else -M % 8, pad if lb == 1 else -N % 8, 0)
            C, cfg = run_gpu(dtype, A, B, la, lb, lc=0, pads=pads, force="%s:s%d" % (tile, slices), return_config=True)
            assert np.array_equal(C.astype(np.float64), ref), (M, N, K, la, lb, slices, cfg, g.last_kernel())


@pytest.mark.parametrize("tile", sorted(TILES))
def test_same_bits_as_the_register_staged_kernel(tile):
    bm, bn, fewest = TILES[tile]
    for M, N, K in ((9 * bm, 8 * bn, 64 * fewest), (bm + 5, 12 * bn - 7, 64 * fewest + 29)):
        A, B = gi.make_problem(M + K, M, N, K, "normal", "f16")
        for la, lb in ((0, 0), (0, 1), (1, 1)):
            pads = (24 + -(K if la == 0 else M) % 8, 40 + -(N if lb == 0 else K) % 8, 0)
            runs, ran = zip(*((run_gpu("f16", A, B, la, lb, pads=pads, force="%s:s1%s" % (tile, how)), g.last_kernel()) for how in ("", ":safe", ":regload")))
            assert ran[:2] == ("gemm_stage_kernel", "gemm_stage_kernel") and ran[2] == "gemm_tile_kernel", ran
            assert np.array_equal(runs[0], runs[1]) and np.array_equal(runs[0], runs[2]), (M, N, K, la, lb)
