"""gemm_f32 computes what binary32 multiply-adds compute, on every tile and whatever the operands hold: edges of tiles and
of K, every bit of an operand over the whole range, products rounded once, nothing from the padding.  (Sums of a few
bfloat16 pieces per operand pass most of this and fail the sums of one product.)"""
import numpy as np
import pytest

import gemm_inputs as gi
from gpu_util import all_tiles, check, run_gpu

pytestmark = pytest.mark.gpu

TILES = ("t256x256", "t128x128", "t256x128", "t128x256", "t64x128", "t128x64")
LAYOUTS = ((0, 0), (0, 1), (1, 0), (1, 1))


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("shape", [(1, 1, 1), (129, 127, 33), (255, 257, 47), (300, 520, 16), (64, 66, 165), (260, 131, 95),
                                   (131, 67, 64), (3, 261, 97), (261, 5, 65), (7, 6, 79)])
def test_edges_of_tiles_and_of_k(oracle, tile, shape):
    M, N, K = shape
    A, B = gi.make_problem(700 + M, M, N, K, "normal", "f32")
    ref = oracle.gemm(M, N, K, A, 0, B, 0, "f32")
    for i, (la, lb) in enumerate(LAYOUTS):
        for splits in (1, 2):
            C = run_gpu("f32", A, B, la, lb, lc=i % 2, pads=(i, 3 - i, 0), force="%s:s%d" % (tile, splits))
            if K >= 16:
                check(C, ref, A, B, "f32", "%s %s %s%s s%d" % (tile, shape, la, lb, splits))
            else:  # a single product
                assert np.all(np.abs(C - ref) <= 2.0 ** -23 * np.abs(ref))


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("low,high", [(-3, 3), (-100, 120), (-149, -120), (120, 127.99), (-109, -103)])
def test_every_bit_of_an_operand_arrives(tile, low, high):
    """A permutation matrix times B is B with its rows permuted, bit for bit: ordinary magnitudes, almost all of
    the range, subnormal numbers, the largest, and numbers just above where three bfloat16 pieces end."""
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
    """Products of ordinary size from operands around 2^-130 and 2^120."""
    rng = np.random.default_rng(9)
    M, N, K = 140, 300, 77
    A = (rng.normal(size=(M, K)) * 2.0 ** -128).astype(np.float32)
    B = (rng.normal(size=(K, N)) * 2.0 ** 120).astype(np.float32)
    ref = oracle.gemm(M, N, K, A, 0, B, 0, "f32")
    for la, lb in LAYOUTS:
        check(run_gpu("f32", A, B, la, lb, force=tile), ref, A, B, "f32", tile)


@pytest.mark.parametrize("tile", all_tiles())
def test_a_sum_of_one_product_is_that_product_rounded_once(oracle, tile):
    """A diagonal matrix with full significands: every entry of C is one product, which binary32 multiply-adds round
    once (the exact product of two binary32 numbers fits binary64)."""
    rng = np.random.default_rng(31)
    for K, N in ((64, 130), (150, 140), (257, 96)):
        d = rng.uniform(1, 2, K).astype(np.float32) * rng.choice((-1, 1), K).astype(np.float32)
        B = rng.normal(size=(K, N)).astype(np.float32)
        want = (d.astype(np.float64)[:, None] * B.astype(np.float64)).astype(np.float32)
        for la, lb in LAYOUTS:
            assert np.array_equal(run_gpu("f32", np.diag(d), B, la, lb, force=tile), want), (tile, K, N, la, lb)
            assert np.array_equal(run_gpu("f32", np.ascontiguousarray(B.T), np.diag(d), la, lb, force=tile), want.T), (tile, K, N, la, lb)


@pytest.mark.parametrize("tile", all_tiles())
def test_padding_of_the_operands_does_not_enter(tile):
    """Elements between the extent and the leading dimension, whatever they hold (whole numbers read as binary32 are
    subnormal; infinities; NaN), leave every bit of C as zeros there do."""
    import torch
    import paper_2003_06324_amd as g
    rng = np.random.default_rng(37)
    M, N, K = 141, 203, 100
    stream = torch.cuda.current_stream().cuda_stream
    for la, lb in LAYOUTS:
        A, B = rng.normal(size=(M, K)).astype(np.float32), rng.normal(size=(K, N)).astype(np.float32)
        results = []
        for filler in (0.0, 7 * 2.0 ** -149, -(2.0 ** -126 - 2.0 ** -149), np.inf, np.nan):
            bufs = []
            for X, lay in ((A, la), (B, lb)):
                rows = X if lay == gi.ROW_MAJOR else X.T
                buf = np.full((rows.shape[0], rows.shape[1] + 11), filler, np.float32)
                buf[:, :rows.shape[1]] = rows
                bufs.append(torch.from_numpy(buf).cuda())
            C = torch.empty((M, N), dtype=torch.float32, device="cuda")
            g.force_config(tile)
            try:
                g.gemm_f32(M, N, K, bufs[0], la, bufs[0].shape[1], bufs[1], lb, bufs[1].shape[1], C, gi.ROW_MAJOR, 0, stream)
            finally:
                g.force_config(None)
            results.append(C.cpu().numpy())
        for C in results[1:]:
            assert np.array_equal(C.view(np.uint32), results[0].view(np.uint32)), (tile, la, lb)


@pytest.mark.parametrize("shape", [(1024, 1024, 2048), (1280, 1280, 1280)])
def test_products_in_one_slice_are_captured_on_a_fresh_stream(shape):
    """Sizes that fill the chip without K slices need no workspace, so the first call on a stream can be recorded into
    a graph."""
    import torch
    import paper_2003_06324_amd as g
    M, N, K = shape
    gen = torch.Generator(device="cuda").manual_seed(3)
    A = torch.randn((M, K), generator=gen, device="cuda")
    B = torch.randn((N, K), generator=gen, device="cuda")
    want = torch.empty((M, N), device="cuda")
    g.force_config(None)
    g.gemm_f32(M, N, K, A, gi.ROW_MAJOR, 0, B, gi.COL_MAJOR, 0, want, gi.ROW_MAJOR, 0, torch.cuda.current_stream().cuda_stream)
    assert g.last_config().split()[4] == "s1"
    C = torch.zeros((M, N), device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        g.gemm_f32(M, N, K, A, gi.ROW_MAJOR, 0, B, gi.COL_MAJOR, 0, C, gi.ROW_MAJOR, 0, torch.cuda.current_stream().cuda_stream)
    for _ in range(3):
        C.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(C, want)
