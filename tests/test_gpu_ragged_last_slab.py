"""The last slab of the tile kernels on direct loads: every kind of remainder of K in a slab, a k-group and a granule,
granules that straddle the end of the operand, leading dimensions below the granule, K-slices."""
import numpy as np
import pytest

import gemm_inputs as gi
from gpu_util import run_gpu

pytestmark = pytest.mark.gpu

TILES = {"t256x256": (256, 256), "t256x256w8": (256, 256), "t256x128": (256, 128), "t128x256": (128, 256), "t128x128": (128, 128),
         "t64x64": (64, 64), "t64x128": (64, 128), "t128x64": (128, 64)}
KS = [1, 3, 4, 9, 20, 31, 63, 65, 136, 191, 202, 448, 517]


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("tile", sorted(TILES))
def test_exact_on_whole_numbers_at_every_remainder(oracle, tile, dtype):
    bm, bn = TILES[tile]
    many = dtype == "f16" and bm * bn <= 128 * 128   # more tiles than CUs: fewer run another kernel in 16 bits
    for n, K in enumerate(KS):
        M, N = (bm + 3, bn - 1) if n % 3 == 0 else ((bm, bn + 6) if n % 3 == 1 else (5, 2))
        if many:
            M, N = ((bm * 17 - 3, bn * 16 - 1), (8 * bm, 33 * bn), (2, 257 * bn))[n % 3]
            K = min(K, 150)
        # (|a|, |b| <= 4: every partial sum is a whole number below 2^24, so any order of summation is exact)
        A, B = gi.make_problem(2300 + K, M, N, K, "int", dtype)
        ref = oracle.gemm(M, N, K, A, 0, B, 0, dtype)
        for la, lb in ((0, 0), (0, 1), (1, 0), (1, 1)) if not many else (((0, 1), (1, 0)) if n % 2 else ((0, 0), (1, 1))):
            # leading dimensions of whole words in 16 bits, so that the direct loads serve them (padding is NaN)
            pads = tuple((x % 2 if dtype == "f16" else 0) + 2 * (n % 2) for x in (K if la == 0 else M, N if lb == 0 else K)) + (0,)
            for slices in (1, 3):
                C, cfg = run_gpu(dtype, A, B, la, lb, lc=0, pads=pads, force="%s:s%d" % (tile, slices), return_config=True)
                assert "aligned" in cfg, cfg
                assert np.array_equal(C.astype(np.float64), ref), (M, N, K, la, lb, slices, cfg)
