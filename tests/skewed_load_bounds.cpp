// Walks the direct loads of gemm_stage_kernel on straightened rows (SKEW) on the CPU, with the kernel's own addresses and rules:
// none reads outside its operand, and every granule of every slab is where the fragments look for it.  Built and run by
// test_skewed_load_bounds.py.
#include "gemm_stage_kernel.h"

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <vector>

using namespace gemm_gfx950;

static long long g_loads = 0, g_wrong = 0;

template <int R> static void walk(int extent, int64_t ld, int K, int per)
{
    typedef _Float16 T;
    typedef StageLoader<T, R, 4, true, true> Loader;
    constexpr int BK = Elem<T>::BK, EPC = Elem<T>::EPC;
    const int64_t last = (extent - 1) * ld + K;  // elements of the operand
    const int KT = (K + BK - 1) / BK;
    for (int row0 = 0; row0 < extent; row0 += R)
        for (int kt0 = 0; kt0 < KT; kt0 += per) {
            const int n = std::min(per, KT - kt0), krem = std::min(K - (kt0 + n - 1) * BK, BK);
            std::vector<int64_t> lds((size_t)(n + 1) * R * GPR, -1);  // element that begins the granule at [image][row][position]
            for (int h = 0; h <= n; ++h)
                for (int i = 0; i < Loader::PER_WAVE; ++i)
                    for (int wave = 0; wave < 4; ++wave)
                        for (int lane = 0; lane < 64; ++lane) {
                            const int r = Loader::ROWS_PER_LOAD * (wave * Loader::PER_WAVE + i) + lane / GPR;
                            const int skew = line_skew(ld, sizeof(T), extent, lane / GPR), g = ((lane % GPR) ^ swz_kc(r)) - skew;
                            if (h >= n - 1 && g * EPC >= krem - (h - (n - 1)) * BK) continue;  // ragged_slab: loads from outside the range
                            const int64_t at = row0 * ld + (int64_t)(kt0 + h) * BK + (Loader::granule(ld, row0, extent, i, wave, lane) - 16 * skew) / 2;
                            ++g_loads;
                            // from two slabs before the end on the range is exact; it drops what reaches past the end
                            if (at < 0 || (h < n - 2 && at + EPC > last)) ++g_wrong;
                            lds[((size_t)h * R + r) * GPR + lane % GPR] = at;
                        }
            for (int t = 0; t < n; ++t)
                for (int r = 0; r < std::min(R, extent - row0); ++r)
                    for (int g = 0; g < GPR; ++g) {
                        const int k = (kt0 + t) * BK + g * EPC, place = g + line_skew(ld, sizeof(T), extent, r & 31);
                        if (k >= K) continue;
                        if (lds[((size_t)(t + place / GPR) * R + r) * GPR + ((place % GPR) ^ swz_kc(r))] != (row0 + r) * ld + k) ++g_wrong;
                    }
        }
}

int main()
{
    for (int extent : {1, 7, 8, 9, 63, 64, 65, 130})
        for (int K : {1, 8, 56, 64, 65, 120, 128, 200, 449})
            for (int64_t pad : {0, 4, 8, 16, 24, 40, 56, 64})
                for (int slices : {1, 2, 3}) {
                    const int KT = (K + 63) / 64;
                    if (slices > KT) continue;
                    walk<64>(extent, (K + 7) / 8 * 8 + pad, K, (KT + slices - 1) / slices);
                    walk<128>(extent, (K + 7) / 8 * 8 + pad, K, (KT + slices - 1) / slices);
                }
    printf("%lld loads, %lld wrong\n", g_loads, g_wrong);
    return g_wrong != 0;
}
