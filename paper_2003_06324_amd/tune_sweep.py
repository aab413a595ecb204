"""Exhaustive sweep of tile configurations and K-slice counts on a list of shapes, the way the
paper tunes its block tile per input size (Section 5.3: powers of two, small sizes up to 1024
and large sizes 1024..4096).  Prints, per shape, the automatic choice, the best forced
configuration and the ratio between the two; the cost model in csrc/gemm_api.hip was
calibrated on this output.

    python3 -m paper_2003_06324_amd.tune_sweep            # default shape list
    python3 -m paper_2003_06324_amd.tune_sweep f16 1536 1024 2048 NT
    python3 -m paper_2003_06324_amd.tune_sweep unaligned  # only the shapes with offset bases
    python3 -m paper_2003_06324_amd.tune_sweep --all      # also print every forced configuration's time
    python3 -m paper_2003_06324_amd.tune_sweep --shapes-file shapes.txt   # lines "f16 M N K NT [offset]"

A shape may carry a byte offset added to both operand bases: operands that are not 16-byte
aligned run the register-staged kernels, and 2-byte aligned ones a slower class of those.
"""
import os
import sys

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

DEFAULT_SHAPES = [
    # benchmark configurations
    ("f32", 256, 256, 256, "NN"), ("f32", 4096, 4096, 4096, "NT"), ("f16", 8192, 8192, 8192, "NT"),
    ("f16", 1000, 1500, 2000, "NN"), ("f16", 4097, 3073, 1025, "NN"), ("f16", 8192, 128, 8192, "TN"),
    ("f16", 128, 8192, 8192, "TN"), ("f16", 1024, 1024, 65536, "TN"),
    # the paper's own sizes: its headline 1536x1024x2048 NT, small (<= 1024) and large (1024..4096)
    ("f16", 1536, 1024, 2048, "NT"), ("f16", 256, 256, 256, "NT"), ("f16", 512, 512, 512, "NT"),
    ("f16", 1024, 1024, 1024, "NT"), ("f16", 2048, 2048, 2048, "NT"), ("f16", 4096, 4096, 4096, "NT"),
    ("f16", 1024, 4096, 2048, "NN"), ("f16", 4096, 1024, 1024, "TT"),
    ("f32", 1024, 1024, 1024, "NT"), ("f32", 2048, 2048, 2048, "NT"),
]
UNALIGNED_SHAPES = [
    ("f16", 2048, 2048, 2048, "NT", 8), ("f16", 2048, 2048, 2048, "NT", 2), ("f16", 2048, 2048, 2048, "TN", 4),
    ("f16", 1024, 1024, 1024, "NT", 2), ("f16", 512, 512, 512, "NT", 8), ("f16", 1536, 1024, 2048, "NT", 8),
    ("f16", 4096, 4096, 1024, "NT", 2), ("f16", 4096, 4096, 4096, "NT", 8),
    ("f32", 2048, 2048, 2048, "NT", 4), ("f32", 1024, 1024, 1024, "NN", 8),
]


def main():
    import torch
    import gemm_inputs as gi
    import paper_2003_06324_amd as g

    show_all = "--all" in sys.argv
    if show_all:
        sys.argv.remove("--all")
    shapes = DEFAULT_SHAPES + UNALIGNED_SHAPES
    if "--shapes-file" in sys.argv:
        i = sys.argv.index("--shapes-file")
        shapes = []
        for line in open(sys.argv[i + 1]):
            f = line.split()
            if f and not f[0].startswith("#"):
                shapes.append((f[0], int(f[1]), int(f[2]), int(f[3]), f[4]) + ((int(f[5]),) if len(f) > 5 else ()))
        del sys.argv[i:i + 2]
    if len(sys.argv) == 2 and sys.argv[1] == "unaligned":
        shapes = UNALIGNED_SHAPES
    if len(sys.argv) >= 6:
        shapes = [(sys.argv[1], int(sys.argv[2]), int(sys.argv[3]), int(sys.argv[4]), sys.argv[5]) +
                  ((int(sys.argv[6]),) if len(sys.argv) > 6 else ())]
    stream = torch.cuda.current_stream().cuda_stream

    def timed(fn, configs, iters, warm=3):
        """Microseconds per call of fn under each forced configuration of `configs` (None: the automatic choice).
        Everything is enqueued back to back, an event pair per configuration, and the host waits once at the end:
        the part lowers its clock within microseconds of idling, so a wait per configuration would time each one
        on a clock that is still rising."""
        pairs = []
        g.force_config(None)
        for _ in range(40):     # brings the part to the shape's steady clock and fills the queue: a launch of a few
            fn()                # microseconds at the head of a short queue is timed at the host's pace
        for cfg in configs:
            g.force_config(cfg)
            for _ in range(warm):
                fn()
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(iters):
                fn()
            e1.record()
            pairs.append((e0, e1))
        g.force_config(None)
        torch.cuda.synchronize()
        return [e0.elapsed_time(e1) / iters * 1e3 for e0, e1 in pairs]

    def us_str(us):
        return "%.2f" % us if us < 10 else "%.1f" % us   # the few-microsecond shapes differ in the second decimal

    worst = 1.0
    for shape in shapes:
        dt, M, N, K, lay = shape[:5]
        off = shape[5] if len(shape) > 5 else 0
        tdt = torch.float16 if dt == "f16" else torch.float32
        A = torch.randn(M * K + 8, device="cuda", dtype=tdt)
        B = torch.randn(K * N + 8, device="cuda", dtype=tdt)
        C = torch.empty(M * N, device="cuda", dtype=torch.float32)
        la, lb = gi.LAYOUTS[lay]
        call = g.gemm_f16f32 if dt == "f16" else g.gemm_f32
        pA, pB = A.data_ptr() + off, B.data_ptr() + off
        fn = lambda: call(M, N, K, pA, la, 0, pB, lb, 0, C, gi.ROW_MAJOR, 0, stream)
        configs = ["%s:s%d" % (tile, s) for tile in g.config_names() for s in (1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16, 20, 24, 28, 32)]
        takes = [timed(fn, configs, 10), timed(fn, configs, 10)]   # two takes: clock noise only adds time
        results = sorted((min(a, b),) + tuple(c.split(":s")) for c, a, b in zip(configs, *takes))
        results = [(us, tile, int(s)) for us, tile, s in results]
        if show_all:
            print("   all: " + " ".join("%s:s%d=%s" % (t_, s_, us_str(us)) for us, t_, s_ in results), flush=True)
        # the automatic choice and the best forced one again, alternating in one pass, in the same thermal state
        # (the first timings of a shape run on a cooler, faster part)
        best_cfg = "%s:s%d" % (results[0][1], results[0][2])
        again = timed(fn, [None, best_cfg, None, best_cfg, None, best_cfg], 20)
        t_auto, t_best = min(again[0::2]), min(again[1::2])
        fn()
        f = g.last_config().split()
        small = f[-1] == "small"   # the kernel for small products, which is not among the forced configurations
        auto_cfg = " ".join(f[:5])
        if "%s:%s" % (f[1], f[4]) == best_cfg and not small:   # one configuration, timed twice
            t_auto = t_best = min(t_auto, t_best)
        best = (t_best, results[0][1], results[0][2])
        worst = max(worst, t_auto / best[0])
        print("%s %dx%dx%d %s%s: auto %s us [%s] | best %s us %s:s%d | auto/best %.2f | %.1f TFLOP/s%s" % (
            dt, M, N, K, lay, " +%dB" % off if off else "", us_str(t_auto), auto_cfg, us_str(best[0]), best[1], best[2], t_auto / best[0],
            2.0 * M * N * K / t_auto / 1e6, " | auto: kernel for small products" if small else ""), flush=True)
    print("worst auto/best ratio: %.2f" % worst)


if __name__ == "__main__":
    main()
