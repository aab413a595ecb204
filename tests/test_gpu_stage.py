"""The tile kernel for launches of at most one workgroup per CU: slab counts around its number of stages, every
remainder of K in a slab, a k-group and a granule, ragged tiles, narrow leading dimensions, K-slices."""
import numpy as np
import pytest

import gemm_inputs as gi
from gpu_util import run_gpu

pytestmark = pytest.mark.gpu

TILES = {"t64x64": (64, 64), "t64x128": (64, 128), "t128x64": (128, 64), "t128x128": (128, 128)}
# (remainders of 1 .. 63 k, whole slabs; from less than one slab to more than any tile has stages)
KS = [1, 2, 8, 9, 17, 63, 64, 72, 129, 191, 200, 256, 321, 449, 1024, 1033]


@pytest.mark.parametrize("tile", sorted(TILES))
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_exact_on_whole_numbers_at_every_remainder(oracle, tile, dtype):
    bm, bn = TILES[tile]
    for n, K in enumerate(KS):
        # (|a|, |b| <= 4: every partial sum is a whole number below 2^24, so any order of summation is exact)
        M, N = ((bm, bn), (bm + 1, 2 * bn - 1), (2, 6), (bm - 8, bn + 8), (2 * bm + 3, 5))[n % 5]
        A, B = gi.make_problem(2100 + K, M, N, K, "int", dtype)
        bits = (gi.bfloat16_bits(A), gi.bfloat16_bits(B)) if dtype == "bf16" else (A, B)
        ref = oracle.gemm(M, N, K, bits[0], 0, bits[1], 0, dtype)
        for i, (la, lb) in enumerate(((0, 0), (0, 1), (1, 0), (1, 1))):
            # leading dimensions rounded up to whole words, so that the direct loads serve them (padding is NaN)
            pads = ((K if la == 0 else M) % 2, (N if lb == 0 else K) % 2 + 2 * (n % 2), 0)
            for slices in (1, 3):
                C, cfg = run_gpu(dtype, A, B, la, lb, lc=0, pads=pads, force="%s:s%d" % (tile, slices), return_config=True)
                assert "aligned" in cfg, cfg
                assert np.array_equal(C.astype(np.float64), ref), (M, N, K, la, lb, slices, cfg)


@pytest.mark.parametrize("tile", sorted(TILES))
def test_same_bits_as_the_register_staged_kernel(tile):
    bm, bn = TILES[tile]
    for M, N, K in ((2 * bm, bn, 1000), (bm + 5, 3 * bn - 7, 1029), (3 * bm, 2 * bn, 2048)):
        A, B = gi.make_problem(M + K, M, N, K, "normal", "f16")
        for la, lb in ((0, 0), (0, 1), (1, 0), (1, 1)):
            pads = ((K if la == 0 else M) % 2, (N if lb == 0 else K) % 2, 0)
            runs = [run_gpu("f16", A, B, la, lb, pads=pads, force="%s:s2%s" % (tile, how)) for how in ("", ":safe", ":regload")]
            assert np.array_equal(runs[0], runs[1]) and np.array_equal(runs[0], runs[2]), (M, N, K, la, lb)
