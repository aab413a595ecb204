// Small products: one round of loads straight into matrix-instruction operands.
//
// A product of a few hundred rows and columns is over in a few microseconds, and what bounds it is how often a
// memory round trip is waited for: the pipelines of the tile kernels fill and drain around a handful of slabs on
// a handful of CUs.  Here a workgroup of sixteen waves computes one 32x32 block of C; the waves share out K, one
// k-group (what a matrix instruction, or four of binary32, consumes) after the other, so the operands
// of the whole block are requested at once by sixteen waves, without LDS, ring or barrier (read word by word: fragment by
// fragment, see FragmentBesideWords).  The sixteen partial blocks meet in LDS and are added in wave order.  Loads need element alignment only, any leading
// dimension, and are guarded at the edges of K (rows past the edges of M and N re-read the last one).
#pragma once
#include "gemm_kernel.h"

namespace gemm_gfx950 {

constexpr int SMALL_WAVES = 16;

__host__ __device__ __forceinline__ uint32_t two_words_shifted(uint32_t hi, uint32_t lo, int bits)
{
#if defined(__HIP_DEVICE_COMPILE__)  // (of the 64-bit shift the compiler makes two instructions, one of them a slow one)
    return __builtin_amdgcn_alignbit(hi, lo, bits);
#else
    return (uint32_t)((((uint64_t)hi << 32) | lo) >> bits);
#endif
}

// Eight 16-bit elements that may begin in the middle of a word, read as the words they begin in and the last element by itself
// (nothing behind it, which may be nobody's), and shifted into place.  What makes the reads is handed in.
struct WordFragment {
    uint4_t w;
    uint32_t last;
    int late;

    template <typename Read> __host__ __device__ __forceinline__ void read(const uint16_t *p, const Read &from)
    {
        late = (int)((uintptr_t)p >> 1) & 1;
        w = from.words(p - late);
        last = from.element(p + 7);
    }
    __host__ __device__ __forceinline__ uint4_t shifted() const
    {
        uint4_t o;
#pragma unroll
        for (int x = 0; x < 4; ++x) o[x] = two_words_shifted(x < 3 ? w[x + 1] : last, w[x], 16 * late);
        return o;
    }
};
struct GlobalRead {
    typedef uint4_t words_t __attribute__((aligned(4)));
    __host__ __device__ __forceinline__ uint4_t words(const uint16_t *p) const { return *(const words_t *)p; }
    __host__ __device__ __forceinline__ uint32_t element(const uint16_t *p) const { return *p; }
};

// The fragment of one k-group: EPL consecutive k of one row, zero from kend on (full: the group lies below kend).
template <typename T, bool KC>
__device__ __forceinline__ typename Frag<T>::type small_fragment(const T *base, int64_t ld, int64_t row, int k, int kend, bool full)
{
    constexpr int EPL = Elem<T>::KG / 2;  // elements per lane
    typedef typename Frag<T>::type frag_t;
    frag_t f;
    if constexpr (KC) {
        typedef frag_t loose_t __attribute__((aligned(sizeof(T))));
        const T *p = base + row * ld + k;
        if (full) {
            f = *(const loose_t *)p;
        } else {
#pragma unroll
            for (int x = 0; x < EPL; ++x) f[x] = k + x < kend ? p[x] : (T)0.0f;
        }
    } else {
        const T *p = base + (int64_t)k * ld + row;
        if (full) {
#pragma unroll
            for (int x = 0; x < EPL; ++x) f[x] = p[(int64_t)x * ld];
        } else {
#pragma unroll
            for (int x = 0; x < EPL; ++x) f[x] = k + x < kend ? p[(int64_t)x * ld] : (T)0.0f;
        }
    }
    return f;
}

// The same in the forms of the kernel where an operand is read word by word.  16-bit rows of an odd leading dimension begin in the
// middle of a word every second time, and 16 bytes from such an address are split up by the memory pipeline, which a product of one
// round of loads waits for (255x255x255 NT 5.0 us, word by word 3.3; 109x451x137 3.1, 2.75).  They are forms of their own: as a choice
// made at run time the words made 427 instructions 876, which rows on words carried along (300x200x136 NT 2.67 us, 2.76).
// WORDS: this operand is the one, and a fragment is waited for before the next one is asked for.  One round of a workgroup's waves
// reads 256 consecutive k, whose lines fill half of the L1 and serve four waves each; with more on the way they are gone before they
// have (1023x255x1151 NT 9.6 us with four groups asked for at once, 8.9 with one, 7.85 with one fragment; K = 137 .. 1023 within 2 %).
// The elements of an operand that is not K-contiguous are put together when all are there.
template <typename T, bool KC, bool WORDS> struct FragmentBesideWords {
    typedef typename Frag<T>::type frag_t;
    static constexpr int EPL = Elem<T>::KG / 2;
    frag_t f;
    uint32_t element[EPL];

    template <bool FULL> __device__ __forceinline__ void read(const T *base, int64_t ld, int64_t row, int k, int kend)
    {
        const uint16_t *const p = (const uint16_t *)base;
        if constexpr (WORDS && FULL) {
            WordFragment words;
            __builtin_amdgcn_sched_barrier(0);
            words.read(p + row * ld + k, GlobalRead());
            f = __builtin_bit_cast(frag_t, words.shifted());
            __builtin_amdgcn_sched_barrier(0);
        } else if constexpr (KC) {
            f = small_fragment<T, KC>(base, ld, row, k, kend, FULL);
        } else {
#pragma unroll
            for (int x = 0; x < EPL; ++x) element[x] = p[(int64_t)(FULL || k + x < kend ? k + x : kend - 1) * ld + row];
        }
    }
    template <bool FULL> __device__ __forceinline__ frag_t get(int k, int kend) const
    {
        if constexpr (KC) return f;
        uint4_t o;
#pragma unroll
        for (int x = 0; x < EPL / 2; ++x)
            o[x] = (FULL || k + 2 * x < kend ? element[2 * x] : 0) | (FULL || k + 2 * x + 1 < kend ? element[2 * x + 1] << 16 : 0);
        return __builtin_bit_cast(frag_t, o);
    }
};

// whether the rows of a K-contiguous operand are read word by word (a base in the middle of a word stays with the loads that read
// nothing in front of it)
template <typename T> bool small_by_words(const void *base, int64_t ld) { return sizeof(T) == 2 && ((uintptr_t)base & 3) == 0 && (ld & 1) != 0; }

// AW, BW: the operand is read word by word
template <typename T, bool AKC, bool BKC, bool AW, bool BW>
__global__ __launch_bounds__(SMALL_WAVES * 64) void gemm_small_kernel(const KernelArgs p)
{
    constexpr int KG = Elem<T>::KG, W = SMALL_WAVES, BATCH = 4;
    constexpr int SW = 33;  // row stride of a partial block in LDS, in words
    typedef typename Frag<T>::type frag_t;
    __shared__ float part[W][32 * SW];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tile_m = blockIdx.x / p.tiles_n, tile_n = blockIdx.x - tile_m * p.tiles_n;
    const int m0 = tile_m * 32, n0 = tile_n * 32;
    const T *A = (const T *)p.A, *B = (const T *)p.B;
    const int m = m0 + (lane & 31) < p.M ? m0 + (lane & 31) : p.M - 1;
    const int n = n0 + (lane & 31) < p.N ? n0 + (lane & 31) : p.N - 1;
    const int groups = (p.K + KG - 1) / KG, kl = (KG / 2) * (lane >> 5);
    static_assert((AKC || !AW) && (BKC || !BW) && (sizeof(T) == 2 || (!AW && !BW)), "words are a matter of K-contiguous 16-bit rows");
    float16_t acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
    const int whole = p.K / KG;
    int g = wave;  // the wave's k-groups are wave, wave + W, ...
    if constexpr (AW || BW) {
        auto group = [&](auto full_tag, int g) {
            constexpr bool FULL = decltype(full_tag)::value;
            const int k = g * KG + kl;
            FragmentBesideWords<T, AKC, AW> fa;
            FragmentBesideWords<T, BKC, BW> fb;
            fa.template read<FULL>(A, p.lda, m, k, p.K);
            fb.template read<FULL>(B, p.ldb, n, k, p.K);
            mma(acc, fa.template get<FULL>(k, p.K), fb.template get<FULL>(k, p.K));
        };
#pragma unroll 1
        for (; g < whole; g += W) group(std::true_type(), g);
        if (whole < groups && whole % W == wave) group(std::false_type(), whole);
    } else {
        // as many as BATCH whole ones are requested together
        auto batch = [&](auto n_tag, int g, bool full) {
            constexpr int N = decltype(n_tag)::value;
            frag_t fa[N], fb[N];
#pragma unroll
            for (int b = 0; b < N; ++b) {
                const int k = (g + b * W) * KG + kl;
                fa[b] = small_fragment<T, AKC>(A, p.lda, m, k, p.K, full);
                fb[b] = small_fragment<T, BKC>(B, p.ldb, n, k, p.K, full);
            }
#pragma unroll
            for (int b = 0; b < N; ++b) mma(acc, fa[b], fb[b]);
        };
        for (; g + (BATCH - 1) * W < whole; g += BATCH * W) batch(std::integral_constant<int, BATCH>(), g, true);
        static_assert(BATCH == 4, "the rest is one to three");
        if (g + 2 * W < whole) batch(std::integral_constant<int, 3>(), g, true);
        else if (g + W < whole) batch(std::integral_constant<int, 2>(), g, true);
        else if (g < whole) batch(std::integral_constant<int, 1>(), g, true);
        if (whole < groups && whole % W == wave) batch(std::integral_constant<int, 1>(), whole, false);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) part[wave][(8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * SW + (lane & 31)] = acc[r];
    __syncthreads();
    const int row = tid >> 5, col = tid & 31;
    float s = part[0][row * SW + col];
#pragma unroll
    for (int w = 1; w < W; ++w) s += part[w][row * SW + col];
    if (m0 + row < p.M && n0 + col < p.N) {
        const int64_t at = (int64_t)(m0 + row) * p.ldc + n0 + col;
        if (p.out16) ((_Float16 *)p.C)[at] = (_Float16)s;
        else p.C[at] = s;
    }
}

// The same for binary32 products of so few elements that 16x16 blocks still fit one round of CUs: four times the
// workgroups, and a wave's sum is a quarter of the matrix-instruction time (two 16x16x4 per 8 k, 32 cycles each, where
// four 32x32x2 take 64 each), which a product this small waits for in the open.  The waves share out K as above, in
// groups of 8 k, so that no wave's sum is longer than there (groups of 16 raise the error of K = 333 and 400 by 3 .. 5 %).
template <bool AKC, bool BKC>
__global__ __launch_bounds__(SMALL_WAVES * 64) void gemm_small16_kernel(const KernelArgs p)
{
    constexpr int KG = Elem<float>::KG, W = SMALL_WAVES, BATCH = 4;  // two k per lane and group
    constexpr int SW = 17;                                           // row stride of a partial block in LDS, in words
    typedef float float2_t __attribute__((ext_vector_type(2)));
    __shared__ float part[W][16 * SW];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tile_m = blockIdx.x / p.tiles_n, tile_n = blockIdx.x - tile_m * p.tiles_n;
    const int m0 = tile_m * 16, n0 = tile_n * 16;
    const float *A = (const float *)p.A, *B = (const float *)p.B;
    const int m = m0 + (lane & 15) < p.M ? m0 + (lane & 15) : p.M - 1;
    const int n = n0 + (lane & 15) < p.N ? n0 + (lane & 15) : p.N - 1;
    const int groups = (p.K + KG - 1) / KG, whole = p.K / KG, kl = 2 * (lane >> 4);

    float4_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
    auto fragment = [&](auto kc_tag, const float *base, int64_t ld, int64_t row, int k, bool full) {
        constexpr bool KC = decltype(kc_tag)::value;
        typedef float2_t loose_t __attribute__((aligned(4)));
        const float *q = KC ? base + row * ld + k : base + (int64_t)k * ld + row;
        float2_t f;
        if (KC && full) {
            f = *(const loose_t *)q;
        } else {
#pragma unroll
            for (int x = 0; x < 2; ++x) f[x] = full || k + x < p.K ? q[KC ? (int64_t)x : (int64_t)x * ld] : 0.0f;
        }
        return f;
    };
    // the wave's k-groups are wave, wave + W, ...; as many as BATCH whole ones are requested together
    auto batch = [&](auto n_tag, int g, bool full) {
        constexpr int N = decltype(n_tag)::value;
        float2_t fa[N], fb[N];
#pragma unroll
        for (int b = 0; b < N; ++b) {
            const int k = (g + b * W) * KG + kl;
            fa[b] = fragment(std::integral_constant<bool, AKC>(), A, p.lda, m, k, full);
            fb[b] = fragment(std::integral_constant<bool, BKC>(), B, p.ldb, n, k, full);
        }
#pragma unroll
        for (int b = 0; b < N; ++b)
#pragma unroll
            for (int t = 0; t < 2; ++t) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[b][t], fb[b][t], acc, 0, 0, 0);
    };
    int g = wave;
    for (; g + (BATCH - 1) * W < whole; g += BATCH * W) batch(std::integral_constant<int, BATCH>(), g, true);
    static_assert(BATCH == 4, "the rest is one to three");
    if (g + 2 * W < whole) batch(std::integral_constant<int, 3>(), g, true);
    else if (g + W < whole) batch(std::integral_constant<int, 2>(), g, true);
    else if (g < whole) batch(std::integral_constant<int, 1>(), g, true);
    if (whole < groups && whole % W == wave) batch(std::integral_constant<int, 1>(), whole, false);
#pragma unroll
    for (int r = 0; r < 4; ++r) part[wave][(4 * (lane >> 4) + r) * SW + (lane & 15)] = acc[r];
    __syncthreads();
    if (tid >= 256) return;
    const int row = tid >> 4, col = tid & 15;
    float s = part[0][row * SW + col];
#pragma unroll
    for (int w = 1; w < W; ++w) s += part[w][row * SW + col];
    if (m0 + row < p.M && n0 + col < p.N) p.C[(int64_t)(m0 + row) * p.ldc + n0 + col] = s;
}

}  // namespace gemm_gfx950
