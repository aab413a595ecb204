"""A last round of tiles that fills at most half of the chip: its tiles are cut into K-slices and summed by a second pass.
Full tiles, tiles at the edges of C, every type of C, misaligned operands, the calls that allocate nothing, graph capture."""
import numpy as np
import pytest

import gemm_inputs as gi
from gpu_util import run_gpu

pytestmark = pytest.mark.gpu

# 17 x 16 tiles of 256 x 256: 16 past the 256 of a full round; 18 x 16 with ragged edges: 32
SHAPES = [(17 * 256, 16 * 256, 1600), (17 * 256 + 3, 16 * 256 - 5, 3211)]


def _sampled(oracle, A, B, dtype, rows, cols):
    if dtype == "bf16":
        A, B = gi.bfloat16_bits(A), gi.bfloat16_bits(B)
    return oracle.gemm(len(rows), len(cols), A.shape[1], np.ascontiguousarray(A[rows]), 0, np.ascontiguousarray(B[:, cols]), 0, dtype)


@pytest.mark.parametrize("dtype,out", [("f16", "f32"), ("f16", "f16"), ("bf16", "f32"), ("f32", "f32")])
@pytest.mark.parametrize("shape", SHAPES)
def test_exact_on_whole_numbers(oracle, shape, dtype, out):
    M, N, K = shape
    if dtype == "f32":
        K //= 2
    # (|a|, |b| <= 4: every partial sum is a whole number below 2^24, so any order of summation is exact)
    A, B = gi.make_problem(2500 + M + K, M, N, K, "int", dtype)
    # rows and columns from every tile row and column, the last ones whole
    rows = np.unique(np.r_[np.arange(0, M, 61), np.arange(M - 64, M)])
    cols = np.unique(np.r_[np.arange(0, N, 59), np.arange(N - 64, N)])
    ref = _sampled(oracle, A, B, dtype, rows, cols)
    for la, lb, force in ((0, 1, "t256x256"), (1, 0, "t256x256w8"), (0, 0, "t256x256")):
        pads = tuple((x % 2 if dtype != "f32" and force == "t256x256" else 0) for x in (K if la == 0 else M, N if lb == 0 else K)) + (3 if lb == 0 else 0,)
        C, cfg = run_gpu(dtype, A, B, la, lb, pads=pads, force=force, return_config=True, out=out)
        assert " tail" in cfg, cfg
        got = C[np.ix_(rows, cols)]
        want = oracle.round_to_half(ref) if out == "f16" else ref
        assert np.array_equal(got.astype(np.float64), np.asarray(want, dtype=np.float64)), (shape, la, lb, cfg)
    C, cfg = run_gpu(dtype, A, B, 0, 1, force="t256x256:s1", return_config=True, out=out)
    assert " tail" not in cfg   # one slice asked for by name
    assert np.array_equal(C[np.ix_(rows, cols)].astype(np.float64), np.asarray(oracle.round_to_half(ref) if out == "f16" else ref, dtype=np.float64))


def test_the_fixed_array_and_streams_without_a_workspace():
    """The entry point that allocates nothing keeps the partial tiles in its fixed array; a stream under capture that has
    no workspace yet runs the tiles whole, and the graph replays to the same product."""
    import torch
    import paper_2003_06324_amd as g
    M, N, K = 17 * 256, 16 * 256, 2048
    gen = torch.Generator(device="cuda").manual_seed(7)
    A = torch.randint(-4, 5, (M, K), device="cuda", generator=gen).half()
    B = torch.randint(-4, 5, (K, N), device="cuda", generator=gen).half()
    ref = A.float() @ B.float()
    C = torch.empty(M, N, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    g.force_config("t256x256")
    try:
        g.gemm_f16f32_noalloc(M, N, K, A, 0, 0, B, 0, 0, C, 0, 0, stream)
        assert " tail" in g.last_config() and "static-scratch" in g.last_config()
        assert torch.equal(C, ref)
        fresh = torch.cuda.Stream()
        graph = torch.cuda.CUDAGraph()
        fresh.wait_stream(torch.cuda.current_stream())
        with torch.cuda.graph(graph, stream=fresh):
            g.gemm_f16f32(M, N, K, A, 0, 0, B, 0, 0, C, 0, 0, torch.cuda.current_stream().cuda_stream)
        assert " tail" not in g.last_config()
        for seed in range(3):
            A.copy_(torch.randint(-4, 5, (M, K), device="cuda", generator=gen))
            C.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(C, A.float() @ B.float())
    finally:
        g.force_config(None)


def test_a_captured_call_leaves_its_streams_workspace_alone():
    """Also where the workspace is large enough: the graph touches A, B and C only, so replays on another stream beside
    sliced calls on the stream it was captured on keep their results."""
    import torch
    import paper_2003_06324_amd as g
    M, N, K = 17 * 256, 16 * 256, 2048
    gen = torch.Generator(device="cuda").manual_seed(11)
    A = torch.randint(-4, 5, (M, K), device="cuda", generator=gen).half()
    B = torch.randint(-4, 5, (K, N), device="cuda", generator=gen).half()
    A2, C2 = -A, torch.empty(M, N, device="cuda")
    ref = A.float() @ B.float()
    C = torch.empty(M, N, device="cuda")
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    g.force_config("t256x256")
    try:
        g.gemm_f16f32(M, N, K, A2, 0, 0, B, 0, 0, C2, 0, 0, side.cuda_stream)   # the workspace grows
        assert " tail" in g.last_config()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            g.gemm_f16f32(M, N, K, A, 0, 0, B, 0, 0, C, 0, 0, side.cuda_stream)
        assert " tail" not in g.last_config(), g.last_config()
        for _ in range(4):
            C.zero_()
            C2.zero_()
            torch.cuda.synchronize()
            with torch.cuda.stream(other):
                graph.replay()
            g.gemm_f16f32(M, N, K, A2, 0, 0, B, 0, 0, C2, 0, 0, side.cuda_stream)
            assert " tail" in g.last_config()
            torch.cuda.synchronize()
            assert torch.equal(C, ref) and torch.equal(C2, -ref)
    finally:
        g.force_config(None)


@pytest.mark.parametrize("force", ["t256x256", "t128x128:s4"])
def test_threads_on_their_own_per_thread_streams_do_not_share_a_workspace(force):
    """hipStreamPerThread (the handle 2) names another stream in every thread: sliced calls of two threads overlap on the GPU."""
    import threading
    import torch
    import paper_2003_06324_amd as g
    M, N, K = (17 * 256, 16 * 256, 2048) if force == "t256x256" else (1024, 1024, 4096)
    gen = torch.Generator(device="cuda").manual_seed(13)
    B = torch.randint(-4, 5, (K, N), device="cuda", generator=gen).half()
    A = [torch.randint(-4, 5, (M, K), device="cuda", generator=gen).half() for _ in range(2)]
    C = [torch.zeros(8, M, N, device="cuda") for _ in range(2)]
    torch.cuda.synchronize()
    g.force_config(force)
    configs = []

    def work(i):
        for c in C[i]:
            g.gemm_f16f32(M, N, K, A[i], 0, 0, B, 0, 0, c, 0, 0, 2)
        configs.append(g.last_config())
        torch.cuda.synchronize()

    try:
        threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
    finally:
        g.force_config(None)
    assert len(configs) == 2 and all(" tail" in c or " s4" in c for c in configs), configs
    for i in range(2):
        ref = A[i].float() @ B.float()
        assert all(torch.equal(c, ref) for c in C[i])
