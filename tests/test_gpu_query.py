"""gemm_query_config_layouts answers with the configuration that a launch picks, wherever 16-byte rows begin: on the cache lines, off
them (packed or padded), or bases off them."""
import random

import numpy as np
import pytest

import paper_2003_06324_amd as g
from gpu_util import run_gpu

pytestmark = pytest.mark.gpu

SHAPES = [(448, 1728, 5888), (192, 704, 5952), (192, 7232, 4736), (4152, 144, 3952), (384, 192, 16384), (2048, 2048, 2048), (1536, 1024, 2048)]


def test_a_launch_picks_what_the_query_answers():
    rng = random.Random(17)
    shapes = SHAPES + [tuple(8 * rng.randrange(12, 200) for _ in range(2)) + (8 * rng.randrange(100, 800),) for _ in range(20)]
    for M, N, K in shapes:
        A, B = np.zeros((M, K), np.float16), np.zeros((K, N), np.float16)
        for la in (g.ROW_MAJOR, g.COL_MAJOR):
            for lb in (g.ROW_MAJOR, g.COL_MAJOR):
                for pads, offs in (((0, 0, 0), (0, 0, 0)), ((8, 24, 0), (0, 0, 0)), ((0, 8, 0), (8, 0, 0))):
                    cfg = run_gpu("f16", A, B, la, lb, pads=pads, offsets=offs, return_config=True)[1].split()
                    assert cfg[1] + ":" + cfg[4] == g.query_config(2, M, N, K, 16, la, lb), (M, N, K, la, lb, pads, offs, cfg)
