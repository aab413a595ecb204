// Host-side launcher shared by the per-tile instantiation files: maps the
// run-time (layout, alignment) choice onto the kernel template's booleans.
#pragma once
#include "gemm_kernel.h"
#include "gemm_ksplit_kernel.h"
#include "gemm_small_kernel.h"
#include "gemm_stage_kernel.h"

#include <tuple>
#include <utility>

namespace gemm_gfx950 {

template <typename Tuple, size_t... I>
static void fill_argv(void **argv, Tuple &vals, std::index_sequence<I...>)
{
    ((argv[I] = (void *)&std::get<I>(vals)), ...);
}

// Enqueues one kernel and returns the status of this launch alone (an error some earlier,
// unrelated runtime call left pending in the calling thread is not picked up, unlike with
// hipGetLastError after a <<<>>> launch).
template <typename... Params, typename... Args>
static hipError_t launch_kernel(void (*kernel)(Params...), dim3 grid, dim3 block, hipStream_t s, Args... args)
{
    std::tuple<Params...> vals(args...);
    void *argv[sizeof...(Params)];
    fill_argv(argv, vals, std::index_sequence_for<Params...>());
    return hipLaunchKernel((const void *)kernel, grid, block, argv, 0, s);
}

template <typename T, int BM, int BN, int WM, int WN, bool AKC, bool BKC>
static hipError_t launch_aligned(bool aligned, dim3 grid, hipStream_t s, const KernelArgs &a)
{
    const dim3 block(WM * WN * 64);
    if (!aligned) return launch_kernel(gemm_tile_kernel<T, BM, BN, WM, WN, AKC, BKC, LOADS_STAGED>, grid, block, s, a);
    if (checks_loads<T>(AKC, BKC, a.M, a.N, a.K)) return launch_kernel(gemm_tile_kernel<T, BM, BN, WM, WN, AKC, BKC, LOADS_CHECKED>, grid, block, s, a);
    return launch_kernel(gemm_tile_kernel<T, BM, BN, WM, WN, AKC, BKC, LOADS_DIRECT>, grid, block, s, a);
}

// akc: A is K-contiguous (row-major); bkc: B is K-contiguous (column-major)
template <typename T, int BM, int BN, int WM, int WN>
hipError_t launch_tile(bool akc, bool bkc, bool aligned, dim3 grid, hipStream_t s, const KernelArgs &a)
{
    if (akc && bkc) return launch_aligned<T, BM, BN, WM, WN, true, true>(aligned, grid, s, a);
    if (akc && !bkc) return launch_aligned<T, BM, BN, WM, WN, true, false>(aligned, grid, s, a);
    if (!akc && bkc) return launch_aligned<T, BM, BN, WM, WN, false, true>(aligned, grid, s, a);
    return launch_aligned<T, BM, BN, WM, WN, false, false>(aligned, grid, s, a);
}

// K split across the waves of the workgroup; the caller passes operands the direct loads serve and a K
// that is a multiple of the slab (`aligned` is part of the common signature and always true here)
template <typename T, int BM, int BN>
hipError_t launch_ksplit(bool akc, bool bkc, bool aligned, dim3 grid, hipStream_t s, const KernelArgs &a)
{
    (void)aligned;
    const dim3 block(256);
    if (akc && bkc) return launch_kernel(gemm_ksplit_kernel<T, BM, BN, true, true>, grid, block, s, a);
    if (akc && !bkc) return launch_kernel(gemm_ksplit_kernel<T, BM, BN, true, false>, grid, block, s, a);
    if (!akc && bkc) return launch_kernel(gemm_ksplit_kernel<T, BM, BN, false, true>, grid, block, s, a);
    return launch_kernel(gemm_ksplit_kernel<T, BM, BN, false, false>, grid, block, s, a);
}

// AW: false where small_by_words has no form for it (binary32, operands that are not K-contiguous)
template <typename T, bool AKC, bool BKC, bool AW>
static hipError_t launch_small_b(bool words_b, dim3 grid, hipStream_t s, const KernelArgs &a)
{
    const dim3 block(SMALL_WAVES * 64);
    if constexpr (BKC && sizeof(T) == 2) {
        if (words_b) return launch_kernel(gemm_small_kernel<T, AKC, BKC, AW, true>, grid, block, s, a);
    }
    return launch_kernel(gemm_small_kernel<T, AKC, BKC, AW, false>, grid, block, s, a);
}

template <typename T, bool AKC, bool BKC>
static hipError_t launch_small_ab(dim3 grid, hipStream_t s, const KernelArgs &a)
{
    const bool words_b = small_by_words<T>(a.B, a.ldb);
    if constexpr (AKC && sizeof(T) == 2) {
        if (small_by_words<T>(a.A, a.lda)) return launch_small_b<T, AKC, BKC, true>(words_b, grid, s, a);
    }
    return launch_small_b<T, AKC, BKC, false>(words_b, grid, s, a);
}

template <typename T>
hipError_t launch_small(bool akc, bool bkc, dim3 grid, hipStream_t s, const KernelArgs &a)
{
    if (akc && bkc) return launch_small_ab<T, true, true>(grid, s, a);
    if (akc && !bkc) return launch_small_ab<T, true, false>(grid, s, a);
    if (!akc && bkc) return launch_small_ab<T, false, true>(grid, s, a);
    return launch_small_ab<T, false, false>(grid, s, a);
}

// binary32, 16x16 blocks; a function template so that only its instantiation file compiles the kernel
template <typename T>
hipError_t launch_small16(bool akc, bool bkc, dim3 grid, hipStream_t s, const KernelArgs &a)
{
    const dim3 block(SMALL_WAVES * 64);
    if (akc && bkc) return launch_kernel(gemm_small16_kernel<true, true>, grid, block, s, a);
    if (akc && !bkc) return launch_kernel(gemm_small16_kernel<true, false>, grid, block, s, a);
    if (!akc && bkc) return launch_kernel(gemm_small16_kernel<false, true>, grid, block, s, a);
    return launch_kernel(gemm_small16_kernel<false, false>, grid, block, s, a);
}

// operands the direct loads serve (`aligned` as above)
template <typename T, int BM, int BN, int NST>
hipError_t launch_stage(bool akc, bool bkc, bool aligned, dim3 grid, hipStream_t s, const KernelArgs &a)
{
    (void)aligned;
    const dim3 block(256);
    if (akc && bkc) return launch_kernel(gemm_stage_kernel<T, BM, BN, 2, 2, NST, true, true, false>, grid, block, s, a);
    if (akc && !bkc) return launch_kernel(gemm_stage_kernel<T, BM, BN, 2, 2, NST, true, false, false>, grid, block, s, a);
    if (!akc && bkc) return launch_kernel(gemm_stage_kernel<T, BM, BN, 2, 2, NST, false, true, false>, grid, block, s, a);
    return launch_kernel(gemm_stage_kernel<T, BM, BN, 2, 2, NST, false, false, false>, grid, block, s, a);
}

// the same for a K-contiguous operand whose rows begin off the cache lines, one stage more
template <typename T, int BM, int BN, int NST>
hipError_t launch_skew(bool akc, bool bkc, bool aligned, dim3 grid, hipStream_t s, const KernelArgs &a)
{
    (void)aligned;
    const dim3 block(256);
    if (akc && bkc) return launch_kernel(gemm_stage_kernel<T, BM, BN, 2, 2, NST, true, true, true>, grid, block, s, a);
    if (akc) return launch_kernel(gemm_stage_kernel<T, BM, BN, 2, 2, NST, true, false, true>, grid, block, s, a);
    return launch_kernel(gemm_stage_kernel<T, BM, BN, 2, 2, NST, false, true, true>, grid, block, s, a);
}

typedef hipError_t (*launch_fn)(bool, bool, bool, dim3, hipStream_t, const KernelArgs &);

#define GEMM_DECLARE_TILE(T, BM, BN, WM, WN) \
    extern template hipError_t launch_tile<T, BM, BN, WM, WN>(bool, bool, bool, dim3, hipStream_t, const KernelArgs &);
#define GEMM_INSTANTIATE_TILE(T, BM, BN, WM, WN) \
    template hipError_t launch_tile<T, BM, BN, WM, WN>(bool, bool, bool, dim3, hipStream_t, const KernelArgs &);
#define GEMM_DECLARE_KSPLIT(T, BM, BN) \
    extern template hipError_t launch_ksplit<T, BM, BN>(bool, bool, bool, dim3, hipStream_t, const KernelArgs &);
#define GEMM_INSTANTIATE_KSPLIT(T, BM, BN) \
    template hipError_t launch_ksplit<T, BM, BN>(bool, bool, bool, dim3, hipStream_t, const KernelArgs &);
#define GEMM_DECLARE_STAGE(T, BM, BN, NST) \
    extern template hipError_t launch_stage<T, BM, BN, NST>(bool, bool, bool, dim3, hipStream_t, const KernelArgs &);
#define GEMM_INSTANTIATE_STAGE(T, BM, BN, NST) \
    template hipError_t launch_stage<T, BM, BN, NST>(bool, bool, bool, dim3, hipStream_t, const KernelArgs &);
#define GEMM_DECLARE_SKEW(T, BM, BN, NST) \
    extern template hipError_t launch_skew<T, BM, BN, NST>(bool, bool, bool, dim3, hipStream_t, const KernelArgs &);
#define GEMM_INSTANTIATE_SKEW(T, BM, BN, NST) \
    template hipError_t launch_skew<T, BM, BN, NST>(bool, bool, bool, dim3, hipStream_t, const KernelArgs &);
#define GEMM_DECLARE_SMALL(T) \
    extern template hipError_t launch_small<T>(bool, bool, dim3, hipStream_t, const KernelArgs &);
#define GEMM_INSTANTIATE_SMALL(T) template hipError_t launch_small<T>(bool, bool, dim3, hipStream_t, const KernelArgs &);

}  // namespace gemm_gfx950
