"""Recorded picks where it is bases on words that let the kernel for small products serve rows of an odd leading dimension: a class of
their own, told by the word "words" in a file."""
import numpy as np
import pytest

import gemm_inputs as gi
import paper_2003_06324_amd as g

M, N, K = 95, 131, 511
LINE = "2 95 131 511 2 2 256 0 "


def _saved(path):
    g.tune_save(path)
    return sorted(ln for ln in open(path).read().split("\n") if ln and not ln.startswith("#"))


def test_the_class_in_a_file(tmp_path):
    f, out = tmp_path / "picks.txt", tmp_path / "saved.txt"
    g.tune_clear()
    try:
        lines = [LINE + "t128x128 1", LINE + "t64x64 1 small words", "2 95 131 512 2 2 256 0 t64x128 2 words", "2 95 131 256 2 2 256 0 t64x64 1 small"]
        f.write_text(lines[0] + "\n" + lines[1] + " # measured\n" + lines[2] + " #\n" + lines[3] + "\n")
        g.tune_load(f)
        assert _saved(out) == sorted(lines)
        g.tune_clear()
        for text in (LINE + "t64x64 1 small", LINE + "t64x64 1 words small", LINE + "t64x64 1 small words words", LINE + "t64x64 1 words2",
                     "2 95 131 256 2 2 256 0 t64x64 1 small words",     # served without words
                     "2 95 131 1153 2 2 256 0 t64x64 1 words", "2 2048 2048 511 2 2 256 0 t64x64 1 words",   # not served with them
                     "2 95 131 511 1 2 256 0 t64x64 1 words", "2 95 131 511 0 2 256 0 t64x64 1 words", "4 95 131 511 2 2 256 0 t64x64 1 words"):
            f.write_text(lines[0] + "\n" + text + "\n")
            assert g.tune_load(f, check=False) == -1, text
            assert _saved(out) == [], text
    finally:
        g.tune_clear()


@pytest.mark.gpu
def test_a_pick_of_one_class_is_none_for_the_other(oracle, tmp_path):
    import torch
    from gpu_util import run_gpu, to_device
    A, B = gi.make_problem(5700, M, N, K, "int", "f16")
    ref = oracle.gemm(M, N, K, A, 0, B, 0, "f16")
    f = tmp_path / "picks.txt"

    def ran(offset):
        C, cfg = run_gpu("f16", A, B, 0, 1, offsets=(offset, offset, 0), return_config=True)
        assert np.array_equal(C.astype(np.float64), ref), cfg
        return cfg.split()[1] + (" small" if cfg.endswith(" small") else "")

    g.force_config(None)
    g.tune_clear()
    try:
        f.write_text(LINE + "t128x128 1\n")
        g.tune_load(f)
        assert (ran(0), ran(1)) == ("t64x64 small", "t128x128")
        # measuring the one class leaves what is recorded for the other
        dA, dB = to_device(gi.store(A, gi.ROW_MAJOR)), to_device(gi.store(B, gi.COL_MAJOR))
        dC = torch.empty(M * N, dtype=torch.float32, device="cuda")
        pick = g.tune(g.KIND_F16F32, M, N, K, dA, gi.ROW_MAJOR, 0, dB, gi.COL_MAJOR, 0, dC, gi.ROW_MAJOR, 0, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert ran(0).split()[0] == pick.split(":")[0] and ran(1) == "t128x128"
        assert len(_saved(tmp_path / "saved.txt")) == 2
        f.write_text(LINE + "t64x128 1 words\n")
        g.tune_load(f)
        assert (ran(0), ran(1)) == ("t64x128", "t128x128")
    finally:
        g.tune_clear()
