"""Small binary32 products in 16x16 blocks: the limits of the choice (K = 192, one block per CU), every remainder of the
blocks and of the groups of 8 k that sixteen waves share out."""
import numpy as np
import pytest

import gemm_inputs as gi
from gpu_util import check, run_gpu

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 192), (16, 16, 191), (17, 15, 193), (256, 256, 256), (255, 249, 271), (1, 4096, 258), (4090, 16, 303), (48, 33, 496), (31, 100, 512),
          (257, 256, 320)]


@pytest.mark.parametrize("shape", SHAPES)
def test_exact_on_whole_numbers(oracle, shape):
    M, N, K = shape
    A, B = gi.make_problem(1700 + M + K, M, N, K, "int", "f32")
    ref = oracle.gemm(M, N, K, A, 0, B, 0, "f32")
    for i, (la, lb) in enumerate(((0, 0), (0, 1), (1, 0), (1, 1))):
        for pads, offs in (((0, 0, 0), (0, 0, 0)), ((1, 3, 2), (1, 0, 3))):
            C, cfg = run_gpu("f32", A, B, la, lb, lc=i % 2, pads=pads, offsets=offs, return_config=True)
            assert cfg.endswith(" small"), cfg
            assert np.array_equal(C.astype(np.float64), ref), (shape, la, lb, pads)


def test_within_the_accumulation_bound(oracle):
    for M, N, K in ((256, 256, 512), (100, 200, 333)):
        A, B = gi.make_problem(K, M, N, K, "normal", "f32")
        C, cfg = run_gpu("f32", A, B, 0, 1, return_config=True)
        check(C, oracle.gemm(M, N, K, A, 0, B, 0, "f32"), A, B, "f32", cfg)
