// Walks the word-wise reads of gemm_small_kernel (16-bit K-contiguous rows of an odd leading dimension) on the CPU, with the
// kernel's own reads: none touches a byte outside the operand, and each lane gets its eight elements.  Built and run by
// test_small_words_bounds.py.
#include "gemm_small_kernel.h"

#include <cstdio>
#include <cstring>
#include <vector>

using namespace gemm_gfx950;

static long long g_reads = 0, g_wrong = 0;

struct Recorder {
    const uint16_t *begin, *end;  // the operand, first element to the one behind its last
    void look(const void *p, size_t bytes) const
    {
        ++g_reads;
        if ((const char *)p < (const char *)begin || (const char *)p + bytes > (const char *)end) ++g_wrong;
    }
    uint4_t words(const uint16_t *p) const
    {
        look(p, 16);
        if ((uintptr_t)p & 3) ++g_wrong;
        return GlobalRead().words(p);
    }
    uint32_t element(const uint16_t *p) const
    {
        look(p, 2);
        return GlobalRead().element(p);
    }
};

int main()
{
    constexpr int KG = Elem<_Float16>::KG;
    for (int rows : {1, 2, 3, 32, 95, 96})
        for (int K : {16, 17, 31, 32, 33, 255, 256, 257, 1151, 1152})
            for (int pad : {0, 1, 2, 3}) {
                const int64_t ld = K + pad;
                if (ld % 2 == 0) continue;
                std::vector<uint32_t> room((size_t)(rows * ld) / 2 + 8, 0xffffffffu);
                uint16_t *const base = (uint16_t *)room.data();
                const Recorder read{base, base + (rows - 1) * ld + K};
                for (int64_t i = 0; i < read.end - read.begin; ++i) base[i] = (uint16_t)(i * 40503 >> 3);
                for (int r = 0; r < rows; ++r)
                    for (int g = 0; g < K / KG; ++g)  // whole k-groups; what is left of K is read element by element
                        for (int half = 0; half < 2; ++half) {
                            const uint16_t *p = base + r * ld + g * KG + half * KG / 2;
                            WordFragment words;
                            words.read(p, read);
                            const uint4_t f = words.shifted();
                            if (memcmp(&f, p, 16) != 0) ++g_wrong;
                        }
            }
    printf("%lld reads, %lld wrong\n", g_reads, g_wrong);
    return g_wrong != 0;
}
