"""gemm_f32 on the tiles that multiply binary32 operands as three bfloat16 pieces each: edges of tiles and of
K, operands whose every bit must arrive, and the operands and results the pieces cannot hold (the tile
is then computed with the binary32 matrix instructions)."""
import numpy as np
import pytest

import gemm_inputs as gi
from gpu_util import check, run_gpu

pytestmark = pytest.mark.gpu

TILES = ("t256x256", "t128x128", "t256x128", "t128x256", "t64x128", "t128x64")
LAYOUTS = ((0, 0), (0, 1), (1, 0), (1, 1))


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("shape", [(1, 1, 1), (129, 127, 33), (255, 257, 47), (300, 520, 16), (64, 66, 165), (260, 131, 95)])
def test_edges_of_tiles_and_of_k(oracle, tile, shape):
    M, N, K = shape
    A, B = gi.make_problem(700 + M, M, N, K, "normal", "f32")
    ref = oracle.gemm(M, N, K, A, 0, B, 0, "f32")
    for i, (la, lb) in enumerate(LAYOUTS):
        for splits in (1, 2):
            C = run_gpu("f32", A, B, la, lb, lc=i % 2, pads=(i, 3 - i, 0), force="%s:s%d" % (tile, splits))
            if K >= 16:
                check(C, ref, A, B, "f32", "%s %s %s%s s%d" % (tile, shape, la, lb, splits))
            else:  # one product of two rounded-to-binary32 operands: off by what the pieces leave out and one rounding
                assert np.all(np.abs(C - ref) <= 2.0 ** -23 * np.abs(ref))


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("low,high", [(-3, 3), (-100, 120), (-149, -120), (120, 127.99)])
def test_every_bit_of_an_operand_arrives(tile, low, high):
    """A permutation matrix times B is B with its rows permuted, bit for bit: ordinary magnitudes, almost all of
    the range, subnormal numbers (which the pieces do not hold) and the largest (which round to infinity)."""
    rng = np.random.default_rng(5)
    K, N = 150, 140
    B = (rng.uniform(1, 2, (K, N)) * 2.0 ** rng.uniform(low, high - 1, (K, N)) * rng.choice((-1, 1), (K, N))).astype(np.float32)
    B[3, 5], B[K - 1, N - 1], B[0, 0] = np.float32(2.0 ** low), 0.0, np.finfo(np.float32).max if high > 127 else 1.0
    perm = rng.permutation(K)
    P = np.eye(K, dtype=np.float32)[perm]
    for la, lb in LAYOUTS:
        C = run_gpu("f32", P, B, la, lb, force=tile)
        assert np.array_equal(C.view(np.uint32) & 0x7fffffff, B[perm].view(np.uint32) & 0x7fffffff), (tile, la, lb)
        assert np.array_equal(C, B[perm])
        C = run_gpu("f32", np.ascontiguousarray(B.T), P, la, lb, force=tile)
        assert np.array_equal(C, B.T @ P), (tile, la, lb)


@pytest.mark.parametrize("tile", ("t256x256", "t128x128", "t64x128"))
def test_tiny_operands_against_huge_ones(oracle, tile):
    """Products of ordinary size from operands around 2^-130 (whose low pieces would be lost) and 2^120."""
    rng = np.random.default_rng(9)
    M, N, K = 140, 300, 77
    A = (rng.normal(size=(M, K)) * 2.0 ** -128).astype(np.float32)
    B = (rng.normal(size=(K, N)) * 2.0 ** 120).astype(np.float32)
    ref = oracle.gemm(M, N, K, A, 0, B, 0, "f32")
    for la, lb in LAYOUTS:
        check(run_gpu("f32", A, B, la, lb, force=tile), ref, A, B, "f32", tile)
