// Walks every direct load of the tile kernels on the CPU, with the kernels' own granule addresses and range rules, and
// reports the furthest byte one reads past the end of its operand.  Built and run by test_direct_load_bounds.py.
#include "gemm_kernel.h"
#include "gemm_stage_kernel.h"

#include <algorithm>
#include <cstdio>

using namespace gemm_gfx950;

static long long g_loads = 0, g_wrong = 0;

// One operand of `extent` rows (tile direction) by K, leading dimension ld, cut into slices of `per` slabs.
template <typename T, int R, int NW, bool KC, bool STAGE>
static void walk(int extent, int64_t ld, int K, int per)
{
    typedef DirectLoader<T, R, NW, KC> Ring;
    typedef StageLoader<T, R, NW, KC> Stage;
    constexpr int BK = Elem<T>::BK;
    const T *const origin = (const T *)(uintptr_t)0x10000000;
    const uint64_t last = (uint64_t)(uintptr_t)(origin + (KC ? (extent - 1) * ld + K : (K - 1) * ld + extent));
    // whole dwords are loaded: of an odd number of 16-bit elements the last one brings the two bytes behind it
    const uint64_t allowed = (last + 3) & ~(uint64_t)3;
    const uint64_t end = Ring::end_of(origin, ld, extent, K);
    const int KT = (K + BK - 1) / BK;
    const bool checks = checks_loads<T>(KC, true, extent, 1, K);  // else the kernel without checks runs
    for (int row0 = 0; row0 < extent; row0 += R)
        for (int kt0 = 0; kt0 < KT; kt0 += per) {
            const int kt1 = std::min(kt0 + per, KT), n = kt1 - kt0;
            const int behind = K - kt1 * BK, krem = behind < 0 ? BK + behind : BK;
            const bool checked = STAGE || (checks && (krem < BK || Ring::reaches_end(ld, row0, extent, behind)));
            for (int h = 0; h < n; ++h) {
                const int k0 = (kt0 + h) * BK;
                const uint64_t base = (uint64_t)(uintptr_t)(KC ? origin + row0 * ld + k0 : origin + k0 * ld + row0);
                const bool exact = checked && h >= n - 2;
                for (int i = 0; i < Ring::PER_WAVE; ++i)
                    for (int wave = 0; wave < NW; ++wave)
                        for (int lane = 0; lane < 64; ++lane) {
                            const uint64_t at = base + (STAGE ? Stage::granule(ld, row0, extent, i, wave, lane) : Ring::granule(ld, row0, extent, i, wave, lane));
                            if (KC && h == n - 1 && krem < BK) {
                                const int j = STAGE ? wave * Ring::PER_WAVE + i : wave + i * NW, r = Ring::ROWS_PER_LOAD * j + lane / GPR;
                                if (((lane % GPR) ^ swz_kc(r)) * Elem<T>::EPC >= krem) continue;  // loads from outside the range
                            }
                            ++g_loads;
                            for (uint64_t dword = at; dword < at + 16; dword += 4) {
                                if (exact && dword + 4 > end) continue;  // dropped by the range check
                                if (dword < (uint64_t)(uintptr_t)origin || dword + 4 > allowed) {
                                    if (++g_wrong <= 10)
                                        printf("%s %s tile %d %s: extent %d ld %lld K %d, slabs %d..%d of %d, slab %d: %lld bytes past the end\n",
                                               sizeof(T) == 4 ? "binary32" : "16 bits", STAGE ? "stage" : "ring", R, KC ? "K-contiguous" : "M/N-contiguous",
                                               extent, (long long)ld, K, kt0, kt1, KT, h, (long long)(dword + 4 - last));
                                }
                            }
                        }
            }
        }
}

template <typename T, int R, int NW, bool STAGE> static void sweep()
{
    constexpr int BK = Elem<T>::BK, EPC = Elem<T>::EPC, EVEN = 4 / (int)sizeof(T);  // leading dimensions are whole words
    for (int extent : {1, 2, 3, EPC - 1, EPC, EPC + 1, R - 3, R, R + 1, R + EPC + 2})
        for (int pad : {0, 1, 2, 3, 5, EPC, EPC + 1})
            for (int slabs : {0, 1, 2, 5})
                for (int rem : {1, 2, 3, 4, 7, 8, 9, BK - 1, BK})
                    for (int slices : {1, 2, 3, 6}) {
                        const int K = slabs * BK + rem, KT = slabs + 1, per = (KT + slices - 1) / slices;
                        if (slices > KT || (extent > EPC + 1 && rem > 3 && rem < BK - 1)) continue;
                        const int mc = (extent + pad + EVEN - 1) / EVEN * EVEN, kc = (K + pad + EVEN - 1) / EVEN * EVEN;
                        walk<T, R, NW, false, STAGE>(extent, mc, K, per);
                        walk<T, R, NW, true, STAGE>(extent, kc, K, per);
                    }
}

int main()
{
    sweep<float, 64, 4, false>();
    sweep<float, 128, 4, false>();
    sweep<float, 256, 8, false>();
    sweep<_Float16, 64, 4, false>();
    sweep<_Float16, 128, 4, false>();
    sweep<_Float16, 256, 4, false>();
    sweep<_Float16, 64, 4, true>();
    sweep<_Float16, 128, 4, true>();
    printf("%lld loads, %lld dwords past the end\n", g_loads, g_wrong);
    return g_wrong != 0;
}
