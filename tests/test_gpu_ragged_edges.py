"""Granules that straddle the edge of an operand, every number of elements they can hold there, in the guarded
slabs of the tile kernels: whole-number inputs, so that every entry of C must be exact; padding is NaN."""
import numpy as np
import pytest

import gemm_inputs as gi
from gpu_util import all_tiles, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,tiles", [("f16", all_tiles()), ("bf16", ("t64x64", "t256x256w8")), ("f32", all_tiles())])
@pytest.mark.parametrize("left", range(1, 9))
def test_every_number_of_elements_at_the_edge(oracle, dtype, tiles, left):
    # extents left, granule + left and a few slabs + left; rows 2-, 4- and 16-byte aligned
    shapes = [(56 + left, 72 + left, 128 + left), (left, 8 + left, 64 + left), (130, 120 + left, left)]
    for s, (M, N, K) in enumerate(shapes):
        A, B = gi.make_problem(900 + 10 * left + s, M, N, K, "int", dtype)
        hA, hB = (gi.bfloat16_bits(A), gi.bfloat16_bits(B)) if dtype == "bf16" else (A, B)
        ref = oracle.gemm(M, N, K, hA, 0, hB, 0, dtype)
        for t, tile in enumerate(tiles):
            for la, lb in ((0, 0), (0, 1), (1, 0), (1, 1)):
                for pads in ((0, 0, 0), (8 - left if left < 8 else 8, t % 3, 1)):
                    C = run_gpu(dtype, A, B, la, lb, pads=pads, offsets=(0, t % 2, 0), force=tile)
                    assert np.array_equal(C.astype(np.float64), ref), (dtype, tile, (M, N, K), la, lb, pads)
