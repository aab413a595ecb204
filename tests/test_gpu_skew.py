"""gemm_stage_kernel on K-contiguous rows that begin off the cache lines: every place of a row in its line, one or both operands,
the fewest slabs, remainders of K, ragged tiles, K-slices down to one slab, streamed operands; and on fewer rows than the
straightening needs.  That the form which straightens ran is read from the phase trace."""
import numpy as np
import pytest

import gemm_inputs as gi
import paper_2003_06324_amd as g
from gpu_util import run_gpu

pytestmark = pytest.mark.gpu

TILES = {"t64x64": (64, 64, 32), "t64x128": (64, 128, 24), "t128x64": (128, 64, 24), "t128x128": (128, 128, 24)}


def _run(dtype, A, B, la, lb, **how):
    """(C, configuration, whether the workgroups' rows were straightened) of a product with a forced configuration"""
    import torch
    trace = torch.zeros((256, 8), dtype=torch.int64, device="cuda")
    g.set_phase_trace(trace, 256)
    try:
        C, cfg = run_gpu(dtype, A, B, la, lb, return_config=True, **how)
    finally:
        g.set_phase_trace(None)
    words = trace[trace[:, 0] != 0][:, 6].tolist()
    assert words and len(set(words)) == 1, words
    return C, cfg, words[0] == 1


@pytest.mark.parametrize("tile", sorted(TILES))
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_exact_on_whole_numbers(oracle, tile, dtype):
    bm, bn, fewest = TILES[tile]
    for n, rem in enumerate((64, 8, 9, 63, 64, 33, 16)):
        slices = 1 + n % 2
        K = 64 * (fewest + n) * slices - 64 + rem
        M, N = ((4 * bm, 9 * bn), (bm + 1, 5 * bn - 3), (1000, 320), (7, 600))[n % 4]
        A, B = gi.make_problem(2300 + K, M, N, K, "int", dtype)
        bits = (gi.bfloat16_bits(A), gi.bfloat16_bits(B)) if dtype == "bf16" else (A, B)
        ref = oracle.gemm(M, N, K, bits[0], 0, bits[1], 0, dtype)
        for la, lb in ((0, 0), (0, 1), (1, 1)):
            # (leading dimensions of 8 (1 + n) elements past whole lines where K is contiguous, whole granules elsewhere; padding is NaN)
            pad = -K % 64 + 8 * (1 + n)
            pads = (pad if la == 0 else -M % 8, pad if lb == 1 else -N % 8, 0)
            C, cfg, straightened = _run(dtype, A, B, la, lb, lc=0, pads=pads, force="%s:s%d" % (tile, slices))
            assert straightened == (lb == 1 or M >= 8), (M, N, K, la, lb, slices, cfg, g.last_kernel())
            assert np.array_equal(C.astype(np.float64), ref), (M, N, K, la, lb, slices, cfg, g.last_kernel())


@pytest.mark.parametrize("tile", sorted(TILES))
@pytest.mark.parametrize("last", [1, 2, 3])
def test_a_last_slice_of_a_few_slabs(tile, last):
    """The other slices have the fewest slabs that are straightened; the last one has fewer than the kernel has stages."""
    bm, bn, fewest = TILES[tile]
    slices = fewest
    for rem in (64, 9):
        K = 64 * (fewest * (slices - 1) + last) - 64 + rem
        A, B = gi.make_problem(2500 + K, bm, bn, K, "int", "f16")
        ref = A.astype(np.float64) @ B.astype(np.float64)   # (whole numbers below 2^24: exact)
        for la, lb in ((0, 0), (0, 1), (1, 1)):
            pad = -K % 64 + 24
            pads = (pad if la == 0 else 0, pad if lb == 1 else 0, 0)
            C, cfg, straightened = _run("f16", A, B, la, lb, pads=pads, force="%s:s%d" % (tile, slices))
            assert straightened and "s%d" % slices in cfg.split(), (K, la, lb, cfg, g.last_kernel())
            assert np.array_equal(C.astype(np.float64), ref), (K, la, lb, cfg)


@pytest.mark.parametrize("tile", sorted(TILES))
def test_same_bits_as_the_register_staged_kernel(tile):
    bm, bn, fewest = TILES[tile]
    for M, N, K in ((9 * bm, 8 * bn, 64 * fewest), (bm + 5, 12 * bn - 7, 64 * fewest + 29)):
        A, B = gi.make_problem(M + K, M, N, K, "normal", "f16")
        for la, lb in ((0, 0), (0, 1), (1, 1)):
            pads = (24 + -(K if la == 0 else M) % 8, 40 + -(N if lb == 0 else K) % 8, 0)
            runs, ran = zip(*((run_gpu("f16", A, B, la, lb, pads=pads, force="%s:s1%s" % (tile, how)), g.last_kernel()) for how in ("", ":safe", ":regload")))
            assert ran[:2] == ("gemm_stage_kernel", "gemm_stage_kernel") and ran[2] == "gemm_tile_kernel", ran
            assert _run("f16", A, B, la, lb, pads=pads, force=tile + ":s1")[2]
            assert np.array_equal(runs[0], runs[1]) and np.array_equal(runs[0], runs[2]), (M, N, K, la, lb)


@pytest.mark.parametrize("tile", sorted(TILES))
def test_one_operand_of_two_and_streamed_operands(tile):
    """Both operands K-contiguous, one of them on 8-byte rows, with its base off the lines, or on lines; operands of more than 28 MiB."""
    bm, bn, fewest = TILES[tile]
    for (M, N, K), cases in (((5 * bm, 6 * bn, 64 * fewest), (((8, 4), (0, 0)), ((4, 8), (0, 0)), ((8, 8), (0, 8)), ((8, 8), (8, 0)), ((8, 0), (0, 0)), ((0, 24), (0, 0)))),
                             ((8 * bm, 12 * bn, (15 << 20) // (8 * bm + 12 * bn) // 64 * 64 + 64), (((8, 8), (0, 0)), ((40, 0), (0, 0))))):
        A, B = gi.make_problem(M + K, M, N, K, "normal", "f16")
        for pads, offsets in cases:
            how = dict(pads=pads + (0,), offsets=offsets + (0,))
            C, cfg, straightened = _run("f16", A, B, 0, 1, force=tile + ":s1", **how)
            assert straightened and g.last_kernel() == "gemm_stage_kernel", (M, N, K, pads, offsets, cfg)
            assert np.array_equal(C, run_gpu("f16", A, B, 0, 1, force=tile + ":s1:regload", **how)), (M, N, K, pads, offsets)
