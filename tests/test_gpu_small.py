"""The kernel for small products: every remainder of the 32x32 blocks and of the k-groups its sixteen waves
share out, all operand types and layouts, misaligned rows, and the limits of the sizes it is chosen for."""
import numpy as np
import pytest

import gemm_inputs as gi
from gpu_util import check, run_gpu

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (31, 33, 7), (32, 64, 8), (33, 31, 15), (65, 40, 17), (100, 95, 129), (64, 32, 255), (40, 72, 257), (256, 1024, 256),
          (300, 200, 136), (8, 500, 250)]


def _ref(oracle, A, B, dtype):
    if dtype == "bf16":
        A, B = gi.bfloat16_bits(A), gi.bfloat16_bits(B)
    return oracle.gemm(A.shape[0], B.shape[1], A.shape[1], A, 0, B, 0, dtype)


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("shape", SHAPES)
def test_small_products_are_exact_on_whole_numbers(oracle, dtype, shape):
    M, N, K = shape
    A, B = gi.make_problem(1300 + M + K, M, N, K, "int", dtype)
    ref = _ref(oracle, A, B, dtype)
    for i, (la, lb) in enumerate(((0, 0), (0, 1), (1, 0), (1, 1))):
        for pads, offs in (((0, 0, 0), (0, 0, 0)), ((1, 3, 2), (1, 0, 3))):
            C, cfg = run_gpu(dtype, A, B, la, lb, lc=i % 2, pads=pads, offsets=offs, return_config=True)
            # (2-byte aligned K-contiguous rows are served up to K = 256)
            assert cfg.endswith(" small") or (K > 256 and "general" in cfg), (dtype, shape, la, lb, pads, cfg)
            assert np.array_equal(C.astype(np.float64), ref), (dtype, shape, la, lb, pads, cfg)
        if dtype == "f16":
            C = run_gpu(dtype, A, B, la, lb, out="f16")
            assert np.array_equal(C.view(np.uint16), oracle.round_to_half(ref).view(np.uint16))


@pytest.mark.parametrize("dtype,limit", [("f16", 768), ("bf16", 768), ("f32", 512)])
def test_the_limits_of_the_choice(oracle, dtype, limit):
    for (M, N, K), small in (((256, 512, limit), True), ((256, 512, limit + 8), False), ((512, 512, limit), True),
                             ((513, 512, limit), False)):
        A, B = gi.make_problem(77 + K, M, N, K, "normal", dtype)
        C, cfg = run_gpu(dtype, A, B, 0, 1, return_config=True)
        assert cfg.endswith(" small") == small, (M, N, K, cfg)
        check(C, _ref(oracle, A, B, dtype), A, B, dtype, cfg)


def test_a_recorded_pick_of_the_kernel_gives_way_to_the_tile_kernels(oracle, tmp_path):
    """What asks for a tile kernel -- the synchronised variant, register-staged loads, a way to store C, the phase
    trace -- gets one, also where a recorded pick names the kernel for small products."""
    import torch
    import paper_2003_06324_amd as g
    M, N, K = 96, 64, 128
    A, B = gi.make_problem(1500, M, N, K, "int", "f32")
    ref = oracle.gemm(M, N, K, A, 0, B, 0, "f32")
    g.force_config(None)
    g.tune_clear()
    picks = tmp_path / "picks.txt"
    picks.write_text("4 96 64 128 0 2 256 1 t64x64 1 small\n4 96 64 128 1 2 256 0 t64x64 1 small\n")
    trace = torch.zeros(8 * 64, dtype=torch.int64, device="cuda")
    try:
        g.tune_load(picks)
        assert run_gpu("f32", A, B, 0, 1, return_config=True)[1].endswith(" small")
        for how in ("auto:safe", "auto:regload", "auto:direct", "auto:staged"):
            C, cfg = run_gpu("f32", A, B, 0, 1, force=how, return_config=True)
            assert " small" not in cfg and np.array_equal(C.astype(np.float64), ref), (how, cfg)
        g.set_phase_trace(trace, 64)
        C, cfg = run_gpu("f32", A, B, 0, 1, return_config=True)
        g.set_phase_trace(None)
        assert " small" not in cfg and np.array_equal(C.astype(np.float64), ref), cfg
        assert int(trace[0]) != 0 and int(trace[5]) >= int(trace[0])
    finally:
        g.set_phase_trace(None)
        g.tune_clear()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("K", [17, 255, 257, 767, 1151])
def test_rows_that_begin_in_the_middle_of_a_word(oracle, dtype, K):
    """Odd leading dimensions of one operand or both, bases on words: read word by word, and up to K = 1152."""
    M, N = 95, 130
    A, B = gi.make_problem(5000 + K, M, N, K, "int", dtype)
    ref = _ref(oracle, A, B, dtype)
    for la, lb in ((0, 0), (0, 1), (1, 0), (1, 1)):
        for odd in ((1, 1), (1, 0), (0, 1)):
            minor = (K if la == 0 else M, N if lb == 0 else K)
            pads = tuple((minor[i] + odd[i]) % 2 for i in (0, 1)) + (0,)
            C, cfg = run_gpu(dtype, A, B, la, lb, pads=pads, return_config=True)
            assert cfg.endswith(" small") and np.array_equal(C.astype(np.float64), ref), (la, lb, odd, cfg)


def test_tuning_leaves_the_choice_on_such_rows_to_the_rule(oracle, tmp_path):
    """A search that finds the kernel fastest there records no pick that a file could not hold; later calls run it all the same."""
    import torch
    import paper_2003_06324_amd as g
    M, N, K = 95, 131, 511
    A, B = gi.make_problem(5600, M, N, K, "int", "f16")
    from gpu_util import to_device
    dA, dB = to_device(gi.store(A, gi.ROW_MAJOR)), to_device(gi.store(B, gi.COL_MAJOR))
    dC = torch.empty(M * N, dtype=torch.float32, device="cuda")
    g.force_config(None)
    g.tune_clear()
    try:
        pick = g.tune(g.KIND_F16F32, M, N, K, dA, gi.ROW_MAJOR, 0, dB, gi.COL_MAJOR, 0, dC, gi.ROW_MAJOR, 0, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert np.array_equal(dC.cpu().numpy().reshape(M, N).astype(np.float64), _ref(oracle, A, B, "f16"))
        picks = str(tmp_path / "picks.txt")
        g.tune_save(picks)
        g.tune_clear()
        g.tune_load(picks)
        cfg = run_gpu("f16", A, B, 0, 1, return_config=True)[1].split()
        assert cfg[1] + ":" + cfg[4] == pick, (pick, cfg)
    finally:
        g.tune_clear()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("K", [16, 256, 768, 1152])
def test_whole_k_groups_on_such_rows(oracle, dtype, K):
    """The last fragment of the last row ends with the operand, in the upper half of a word or the lower one."""
    for M, N in ((96, 130), (95, 33)):
        A, B = gi.make_problem(5100 + K, M, N, K, "int", dtype)
        ref = _ref(oracle, A, B, dtype)
        for la, lb in ((0, 0), (0, 1), (1, 0), (1, 1)):
            minor = (K if la == 0 else M, N if lb == 0 else K)
            C, cfg = run_gpu(dtype, A, B, la, lb, pads=(1 + minor[0] % 2, 1 + minor[1] % 2, 0), return_config=True)
            assert cfg.endswith(" small") and np.array_equal(C.astype(np.float64), ref), (M, la, lb, cfg)
