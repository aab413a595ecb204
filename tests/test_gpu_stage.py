"""The tile kernel for launches of at most one workgroup per CU: slab counts around its number of stages, every
remainder of K in a slab, a k-group and a granule, ragged tiles, narrow leading dimensions, K-slices."""
import numpy as np
import pytest

import gemm_inputs as gi
import paper_2003_06324_amd as g
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
                assert "aligned" in cfg and (K % 64 == 0 or g.last_kernel() == "gemm_stage_kernel"), (cfg, g.last_kernel())
                assert np.array_equal(C.astype(np.float64), ref), (M, N, K, la, lb, slices, cfg)


# whole slabs of operands that do not stay in the L2s: the fewest slabs it takes, and each number of them modulo its stages
@pytest.mark.parametrize("tile", sorted(TILES))
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_exact_on_whole_slabs(oracle, tile, dtype):
    bm, bn = TILES[tile]
    fewest = 24 if tile == "t128x128" else 16
    for n in range(7):
        slices = 1 + n % 2
        K = 64 * ((fewest + n) * slices - n % 2)   # two slices: the second one slab shorter
        M, N = ((9 * bm, 14 * bn), (600, 744), (1000, 320), (8, 1400))[n % 4]   # (whole tiles, and whole granules over their edges)
        assert (M + N) * K * 2 >= 5 << 19
        A, B = gi.make_problem(2200 + K, M, N, K, "int", dtype)
        bits = (gi.bfloat16_bits(A), gi.bfloat16_bits(B)) if dtype == "bf16" else (A, B)
        ref = oracle.gemm(M, N, K, bits[0], 0, bits[1], 0, dtype)
        for la, lb in ((0, 0), (0, 1), (1, 0), (1, 1)):
            C, cfg = run_gpu(dtype, A, B, la, lb, lc=0, pads=(8 * (n % 2), 4 * (n % 3), 0), force="%s:s%d" % (tile, slices), return_config=True)
            assert cfg.endswith(" s%d" % slices) and g.last_kernel() == "gemm_stage_kernel", (cfg, g.last_kernel())
            assert np.array_equal(C.astype(np.float64), ref), (M, N, K, la, lb, slices, cfg)


def test_where_it_runs():
    """The limits of the choice: workgroups, slabs, bytes of the operands, granules over an edge; never in binary32 or on
    2-byte aligned rows."""
    def ran(M, N, K, dtype="f16", force="t64x64:s1", pad=0, lb=1):
        A, B = np.zeros((M, K), np.float32 if dtype == "f32" else np.float16), np.zeros((K, N), np.float32 if dtype == "f32" else np.float16)
        run_gpu(dtype, A, B, 0, lb, pads=(pad, pad, 0), force=force)
        return g.last_kernel() == "gemm_stage_kernel"
    assert ran(1024, 1024, 1024) and not ran(1024, 1088, 1024)           # 256 workgroups, 272
    assert not ran(1024, 1024, 960) and ran(1024, 1024, 968)             # 15 slabs; the ragged 16th
    assert not ran(640, 600, 1024) and ran(640, 648, 1024)               # 2.42 MiB, 2.52
    assert ran(256, 256, 28600) and not ran(256, 256, 28736)             # 27.9 MiB, 28.1
    assert not ran(1024, 1024, 1024, "f32") and not ran(1024, 1024, 1024, pad=1)
    assert not ran(512, 512, 2048, force="t256x256:s1")                  # no such kernel for the tile
    big = dict(force="t128x128:s1")                                      # 240 workgroups, 256; the second on 8-byte rows
    assert ran(1920, 2048, 1536, **big) and not ran(2048, 2048, 1536, **big) and ran(2048, 2048, 1536, pad=4, **big)
    assert not ran(640, 596, 448, pad=4, lb=0) and ran(640, 596, 512, pad=4, lb=0) and not ran(640, 600, 512, pad=4, lb=0)


@pytest.mark.parametrize("tile", sorted(TILES))
def test_same_bits_as_the_register_staged_kernel(tile):
    bm, bn = TILES[tile]
    for M, N, K in ((2 * bm, bn, 1000), (bm + 5, 3 * bn - 7, 1029), (7 * bm, 9 * bn, 3072)):
        A, B = gi.make_problem(M + K, M, N, K, "normal", "f16")
        for la, lb in ((0, 0), (0, 1), (1, 0), (1, 1)):
            pads = ((K if la == 0 else M) % 2, (N if lb == 0 else K) % 2, 0)
            runs, ran = zip(*((run_gpu("f16", A, B, la, lb, pads=pads, force="%s:s2%s" % (tile, how)), g.last_kernel()) for how in ("", ":safe", ":regload")))
            assert ran == ("gemm_stage_kernel", "gemm_stage_kernel", "gemm_tile_kernel")
            assert np.array_equal(runs[0], runs[1]) and np.array_equal(runs[0], runs[2]), (M, N, K, la, lb)


@pytest.mark.parametrize("M,N,K", [(120, 3064, 6144), (3072, 128, 6176)])
def test_one_row_or_column_of_tiles_on_streamed_operands(M, N, K):
    """Operands of more than 28 MiB, 96 workgroups, 24 slabs or 25 each."""
    A, B = gi.make_problem(M + K, M, N, K, "normal", "f16")
    assert (M + N) * K * 2 > 28 << 20
    for la, lb in ((0, 0), (0, 1), (1, 0), (1, 1)):
        runs, ran = zip(*((run_gpu("f16", A, B, la, lb, force="t128x128:s4" + how), g.last_kernel()) for how in ("", ":regload")))
        assert ran == ("gemm_stage_kernel", "gemm_tile_kernel")
        assert np.array_equal(runs[0], runs[1]), (la, lb)
    zeros = np.zeros((128, 8192), np.float16), np.zeros((8192, 8192), np.float16)
    run_gpu("f16", *zeros, 0, 1, force="t128x128:s4")                    # a full chip of one row; its rows straightened
    assert g.last_kernel() == "gemm_tile_kernel"
    run_gpu("f16", *zeros, 0, 1, pads=(8, 8, 0), force="t128x128:s4")
    assert g.last_kernel() == "gemm_stage_kernel"
