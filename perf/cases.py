"""Matrix products that a user of this library has it do, as cases to be timed and compared.

Every case is one call of one public entry point, C = A*B with operands already in device memory, as a
program that owns its buffers makes it.  The listed cases are the library's benchmark configurations, the
paper's headline size and small sizes of the tests; draw() covers the ranges around them: all entry points,
all layouts, packed and padded leading dimensions, multiples of 64 and of 8 and odd extents.
"""
import math

import torch

import paper_2003_06324_amd as g

ROW, COL = "row", "col"
LAYOUT = {ROW: g.ROW_MAJOR, COL: g.COL_MAJOR}

# entry point, operand type, type of C
KINDS = {
    "f32": (g.gemm_f32, torch.float32, torch.float32),
    "f16f32": (g.gemm_f16f32, torch.float16, torch.float32),
    "f16f16": (g.gemm_f16f16, torch.float16, torch.float16),
    "bf16f32": (g.gemm_bf16f32, torch.bfloat16, torch.float32),
    "f16f32_noalloc": (g.gemm_f16f32_noalloc, torch.float16, torch.float32),
}

# the largest listed products: binary32 4096^3, 16-bit 8192^3
MOST_FLOPS = {"f32": 2.0 * 4096 ** 3, "16": 2.0 * 8192 ** 3}
MOST_BYTES = 600e6


def _case(name, kind, M, N, K, a, b, c=ROW, pad=0, dist="normal"):
    return {"name": name, "kind": kind, "M": M, "N": N, "K": K, "a": a, "b": b, "c": c, "pad": pad, "dist": dist}


def listed():
    return [
        # a small product inside a larger computation: the latency of one call
        _case("f32_256", "f32", 256, 256, 256, ROW, ROW, dist="uniform"),
        # small and ragged, half-precision result, C stored column by column (a Fortran-style caller)
        _case("f16f16_small_ragged", "f16f16", 300, 200, 136, ROW, COL, COL, dist="uniform"),
        # ordinary single-precision product
        _case("f32_1024", "f32", 1024, 1024, 1024, ROW, COL, dist="uniform"),
        # large single-precision product (benchmark configuration)
        _case("f32_4096", "f32", 4096, 4096, 4096, ROW, COL, dist="uniform"),
        # ordinary sizes that are no multiples of a tile, rows 8-byte aligned (benchmark configuration)
        _case("f16_edge_even", "f16f32", 1000, 1500, 2000, ROW, ROW, dist="uniform"),
        # odd sizes: every second row starts off a 4-byte boundary (benchmark configuration)
        _case("f16_edge_odd", "f16f32", 4097, 3073, 1025, ROW, ROW, dist="uniform"),
        # the paper's headline half-precision size
        _case("f16f16_paper", "f16f16", 1536, 1024, 2048, ROW, COL),
        # ordinary square product in bfloat16, the training dtype
        _case("bf16_2048", "bf16f32", 2048, 2048, 2048, ROW, ROW),
        # tall and thin product (benchmark configuration)
        _case("f16_skinny_n", "f16f32", 8192, 128, 8192, COL, ROW),
        # short and wide product in a serving loop that may not allocate (benchmark configuration)
        _case("f16_skinny_m_noalloc", "f16f32_noalloc", 128, 8192, 8192, COL, ROW),
        # long sum, as in a weight gradient (benchmark configuration)
        _case("f16_deep_k", "f16f32", 1024, 1024, 65536, COL, ROW),
        # the headline benchmark
        _case("f16_8192", "f16f32", 8192, 8192, 8192, ROW, COL),
    ]


def _size(rng, lo, hi, step):
    x = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(hi, max(lo, int(round(x / step)) * step)) if step > 1 else int(round(x))


def draw(rng):
    while True:
        kind = rng.choice(("f32", "f16f32", "f16f32", "f16f16", "bf16f32", "f16f32_noalloc"))
        step = rng.choice((1, 8, 64))  # odd extents, whole 16-byte granules, whole tiles
        family = rng.choice(("small", "ordinary", "ordinary", "skinny", "deep", "large"))
        if family == "small":
            M, N, K = (_size(rng, 64, 512, step) for _ in range(3))
        elif family == "ordinary":
            M, N, K = (_size(rng, 512, 4096, step) for _ in range(3))
        elif family == "skinny":
            M, N, K = _size(rng, 64, 256, step), _size(rng, 2048, 8192, step), _size(rng, 1024, 8192, step)
            if rng.random() < 0.5:
                M, N = N, M
        elif family == "deep":
            M, N, K = _size(rng, 256, 1024, step), _size(rng, 256, 1024, step), _size(rng, 8192, 65536, step)
        else:
            M, N, K = (_size(rng, 4096, 8192, step) for _ in range(3))
        case = _case(family, kind, M, N, K, rng.choice((ROW, COL)), rng.choice((ROW, COL)), rng.choice((ROW, ROW, COL)),
                     rng.choice((0, 0, 8)), rng.choice(("normal", "uniform")))
        del case["name"]
        w = work(case)
        if w["flops"] <= MOST_FLOPS["f32" if kind == "f32" else "16"] and w["bytes"] <= MOST_BYTES:
            return case


def _matrix(rows, cols, layout, pad, dtype, dist, gen):
    """(buffer, leading dimension) of a random rows x cols matrix."""
    major, minor = (rows, cols) if layout == ROW else (cols, rows)
    ld = minor + pad
    x = torch.empty(major * ld, dtype=torch.float32, device="cuda")
    x = x.normal_(generator=gen) if dist == "normal" else x.uniform_(-1.0, 1.0, generator=gen)
    return x.to(dtype), ld


def prepare(case, seed):
    fn, dtype, ctype = KINDS[case["kind"]]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    M, N, K = case["M"], case["N"], case["K"]
    A, lda = _matrix(M, K, case["a"], case["pad"], dtype, case["dist"], gen)
    B, ldb = _matrix(K, N, case["b"], case["pad"], dtype, case["dist"], gen)
    C = torch.zeros((M, N) if case["c"] == ROW else (N, M), dtype=ctype, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    args = (M, N, K, A, LAYOUT[case["a"]], lda, B, LAYOUT[case["b"]], ldb, C, LAYOUT[case["c"]], 0, stream)
    return {"fn": fn, "args": args, "C": C}


def run(state):
    state["fn"](*state["args"])
    return state["C"]


def work(case):
    M, N, K = case["M"], case["N"], case["K"]
    esz = 4 if case["kind"] == "f32" else 2
    csz = 2 if case["kind"] == "f16f16" else 4
    return {"bytes": (M * K + K * N) * esz + M * N * csz, "flops": 2.0 * M * N * K}


def tolerance(case):
    # Four times what the library was seen to differ by from float64 sums of the same operands over the listed and ten
    # drawn cases (2-norm; largest over the root mean square): binary32 operands 1.2e-6; 9.5e-6, 16-bit operands 5.8e-7;
    # 5.1e-6.  Binary16 C, against the float64 sum rounded to it: 1.2e-5, and single elements one step (2^-10) off where
    # the sum lies near the middle between two neighbours.
    if case["kind"] == "f16f16":
        return {"rel": 5e-5, "max": 2e-3}
    if case["kind"] == "f32":
        return {"rel": 5e-6, "max": 4e-5}
    return {"rel": 2.5e-6, "max": 2e-5}


def exact(case, seed):
    """The product of the same operands in binary64, laid out as run() returns it."""
    dtype = KINDS[case["kind"]][1]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    M, N, K = case["M"], case["N"], case["K"]

    def dense(rows, cols, layout):
        x, ld = _matrix(rows, cols, layout, case["pad"], dtype, case["dist"], gen)
        major, minor = (rows, cols) if layout == ROW else (cols, rows)
        x = x.view(major, ld)[:, :minor].to(torch.float64)
        return x if layout == ROW else x.t()

    A = dense(M, K, case["a"])
    B = dense(K, N, case["b"])
    C = torch.matmul(A, B)
    return C if case["c"] == ROW else C.t().contiguous()
