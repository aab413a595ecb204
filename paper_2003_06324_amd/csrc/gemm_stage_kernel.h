// Tile kernel for launches of at most one workgroup per CU (16-bit operands, direct loads).
//
// With a CU to itself a small tile is bound by round trips, not by rates: gemm_tile_kernel fetches the operands of a
// k-group from LDS one k-group (two MFMAs of a 64x128 tile) before they are used, and one of its two operands from
// memory one slab before, so a slab takes 0.38 us whatever the tile (1536x1024x2048, 64x64 .. 128x128, also on
// all-zero operands) where its direct loads alone take 0.19 (24 KB at the 127 GB/s a CU takes such loads) and its
// MFMAs 0.11.  Here
//   - LDS holds NST whole slabs (stages) of both operands, so loads are NST - 2 slabs ahead of their use;
//   - a wave has the fragments of a whole slab in registers and reads those of a k-group of slab t+1 as soon as the MFMAs
//     of that k-group of slab t have been issued: no MFMA waits for an LDS read.
// Per slab t: its MFMAs; meanwhile the reads of slab t+1 and the direct loads of slab t+NST-1 into the slot of slab t-1
// (every wave has multiplied slab t-1, so its reads are done); then one counted wait (slab t+2 landed) and one barrier.
//
// One wave per SIMD issues about one instruction per four to five cycles, so the loop is kept short: the loads of a wave
// are contiguous in LDS and share one M0 value (the instruction offset moves both addresses), fragment addresses are
// registers that move from slot to slot.  Code that runs once costs an instruction-cache miss per 64 bytes, so there is
// one body with loads, one without for the slabs whose successors are all on the way, and the last slab.
//
// Loads are range-checked by their buffer descriptors.  Towards the end of the slice the range is the exact end of the
// operand: k-rows past K, and the part of a granule past the operand's last row, read as zeros.  A ragged last slab
// therefore runs through the same loop: lanes whose whole granule of a K-contiguous operand lies past K load from outside
// the range, the granule that straddles K is masked in registers, and the k-groups past K are skipped.
//
// SKEW: rows of a K-contiguous operand that begin off a 128-byte line.  A row's 128 bytes of a slab then lie in two lines,
// and the second one is fetched again with the next slab (the L1 has long lost it), so the loads cost up to twice the
// lines.  Instead, image s of such an operand holds for every row the s-th whole line from the one on that the row begins
// in; granule j of slab t is then granule (j + d) % 8 of image t + (j + d) / 8, with d = 0 .. 7 the row's place in its
// first line.  That is an address per lane, nothing more, but a slab takes two images, so there is one image more than
// slabs, and one stage more for loads as far ahead.  The loads alone of a 64x128 tile (operands in the memory-side cache)
// take 0.23 us a slab on rows that begin on lines, 0.36 with rows 16 bytes off them; the product 1536x1024x2048, both
// operands K-contiguous and their rows padded by 16 bytes, 17.4 us before and 14.4 with this.
#pragma once
#include "gemm_kernel.h"

namespace gemm_gfx950 {

// Place of row r of a K-contiguous operand in its first line, in granules, counted from the operand's beginning (on a line, where
// it is to pay).  With rows that begin on 16 bytes, eight rows further it is the same again, so it is one number for all rows a
// lane deals with.  Zero where rows do not begin on 16 bytes, and where there are less than the eight rows that the granules in
// front of a row are sure to lie in.
__host__ __device__ __forceinline__ int line_skew(int64_t ld, int esz, int rows, int r)
{
    return ld * esz % 16 != 0 || rows < GPR ? 0 : (int)((uint32_t)r * (uint32_t)(ld * esz / 16) & (GPR - 1));
}

// Direct loads of one operand: the same LDS image as DirectLoader's, wave w filling PER_WAVE consecutive pieces of 1 KiB.
template <typename T, int R, int NW, bool KC, bool SKEW = false>
struct StageLoader {
    static constexpr int EPC = Elem<T>::EPC, BK = Elem<T>::BK;
    static constexpr int PER_WAVE = R * RBK / 1024 / NW;
    static_assert(PER_WAVE >= 1 && R * RBK % (1024 * NW) == 0, "tile too small for this wave count");
    static constexpr int CPR = R / EPC;             // granules per k-row (M/N-contiguous image)
    static constexpr int ROWS_PER_LOAD = 1024 / RBK;
    static constexpr int GROUP = 4;                 // loads per M0 value: the instruction offset is below 4096
    static constexpr int LEAD = (GROUP - 1) * 1024 + (SKEW ? RBK : 0);  // the descriptor's base lies this far before the slab, so
                                                    // that the lane offsets, from which the instruction offset is taken off, stay positive
    int4_t rsrc;
    uint32_t off[PER_WAVE];
    int64_t step;   // bytes to advance per slab
    uint64_t end;   // address of the operand's end
    int skew;       // line_skew of the lane's rows

    // byte offset from the slab's origin of the granule a lane fetches with its wave's load i
    static __host__ __device__ __forceinline__ int64_t granule(int64_t ld, int row0, int rmax, int i, int wave, int lane)
    {
        const int j = wave * PER_WAVE + i;
        if (KC) {
            const int r = ROWS_PER_LOAD * j + lane / GPR;
            const int g = (lane % GPR) ^ swz_kc(r);
            return ((int64_t)(row0 + r < rmax ? r : rmax - 1 - row0) * ld + g * EPC) * (int64_t)sizeof(T);  // rows past the edge re-read the last one
        }
        const int q = 64 * j + lane;
        const int kk = q / CPR;
        const int m = ((q % CPR) ^ swz_mc<T, CPR>(kk)) * EPC;
        return ((int64_t)kk * ld + (row0 + m < rmax ? m : 0)) * (int64_t)sizeof(T);  // granules past the edge re-read the first one
    }
    // kmax: the operand's extent in k (of the whole operand, not of this K-slice); the rest as DirectLoader::init
    __device__ __forceinline__ void init(const T *origin, int64_t ld, int row0, int rmax, int kmax, int k0, int wave, int lane)
    {
        const uint64_t base = (uint64_t)(uintptr_t)(KC ? origin + (int64_t)row0 * ld + k0 : origin + (int64_t)k0 * ld + row0) - LEAD;
        rsrc[0] = (int)(uint32_t)base;
        rsrc[1] = (int)(uint32_t)(base >> 32) & 0xffff;
        rsrc[2] = 0x7fffffff;
        rsrc[3] = 0x00020000;
#pragma unroll
        for (int i = 0; i < PER_WAVE; ++i) off[i] = (uint32_t)granule(ld, row0, rmax, i, wave, lane) + LEAD - i % GROUP * 1024;
        skew = 0;
        if constexpr (SKEW && KC) {
            skew = line_skew(ld, sizeof(T), rmax, lane / GPR);
#pragma unroll
            for (int i = 0; i < PER_WAVE; ++i) off[i] -= 16 * skew;
        }
        step = (KC ? (int64_t)BK : (int64_t)BK * ld) * (int64_t)sizeof(T);
        end = DirectLoader<T, R, NW, KC>::end_of(origin, ld, rmax, kmax);
    }
    // load i of this wave to wave_dst + i KiB (LDS address); with i in order, M0 is set by the first of a group
    __device__ __forceinline__ void issue(uint32_t wave_dst, int i) const
    {
        if (i % GROUP == 0)
            asm volatile("s_add_i32 m0, %0, %1\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %3, 0 offen lds"
                         : : "s"(wave_dst), "i"(i * 1024), "v"(off[i]), "s"(rsrc) : "memory", "m0", "scc");
        else
            asm volatile("buffer_load_dwordx4 %0, %1, 0 offen offset:%2 lds"
                         : : "v"(off[i]), "s"(rsrc), "i"(i % GROUP * 1024) : "memory");
    }
    __device__ __forceinline__ void advance()
    {
        const uint64_t base = (((uint64_t)(uint32_t)rsrc[1] << 32) | (uint32_t)rsrc[0]) + step;
        rsrc[0] = (int)(uint32_t)base;
        rsrc[1] = (int)(uint32_t)(base >> 32);
    }
    // the present slab's range ends with the operand
    __device__ __forceinline__ void exact_range()
    {
        const uint64_t left = end - (((uint64_t)(uint32_t)rsrc[1] << 32) | (uint32_t)rsrc[0]);
        const int range = (left >> 31) != 0 ? 0x7fffffff : (int)(uint32_t)left;
        rsrc[2] = __builtin_amdgcn_readfirstlane(range);  // (uniform anyway, which the compiler does not see through the loop)
    }
    // the present image lies past the slice: nothing is loaded
    __device__ __forceinline__ void no_range() { rsrc[2] = 0; }
    // before the loads of a slab (or image) of which only `krem` k (skewed: from the row's beginning in it on, none or less if the
    // image is past the slice's last slab) lie inside the operand
    __device__ __forceinline__ void ragged_slab(int krem, int wave, int lane)
    {
        if (!KC) return;  // k-rows past K lie past the operand's end
#pragma unroll
        for (int i = 0; i < PER_WAVE; ++i) {
            const int r = ROWS_PER_LOAD * (wave * PER_WAVE + i) + lane / GPR;
            const int g = ((lane % GPR) ^ swz_kc(r)) - skew;
            if (g * EPC >= krem) off[i] = 0x80000000u;
        }
    }
};

// LDS addresses of a wave's fragments of one operand (NF blocks of 32 tile rows from r0 on; see Fetch), as registers that
// move with the slot.  K-contiguous image: one per k-group, the blocks 32 rows apart; M/N-contiguous: one per block, the
// k-groups 16 k-rows apart.
template <typename T, int R, bool KC, int NF, bool SKEW>
struct StageFragments {
    typedef typename Frag<T>::type frag_t;
    static constexpr int NA = KC ? KGS : NF;
    uint32_t at[NA];
    bool next[NA];  // skewed: the granule is in the image behind the slab's own

    // stage: bytes from an image to the one behind it
    __device__ __forceinline__ void init(uint32_t img, int r0, int lane, int64_t ld, int rows, int stage)
    {
#pragma unroll
        for (int x = 0; x < NA; ++x) {
            next[x] = false;
            if (KC) {
                const int r = r0 + (lane & 31);
                int g = 2 * x + (lane >> 5);
                if constexpr (SKEW) {
                    g += line_skew(ld, sizeof(T), rows, lane & 31);
                    next[x] = g >= GPR;
                    g &= GPR - 1;
                }
                at[x] = img + (next[x] ? stage : 0) + r * RBK + ((g ^ swz_kc(r)) << 4);
            } else {
                const int s = lane & 15;
                const int col = r0 + x * 32 + 16 * ((lane >> 4) & 1) + 4 * (s & 3);
                const int kl = 8 * (lane >> 5) + (s >> 2);
                at[x] = img + kl * (R * 2) + (((col >> 3) ^ swz_mc<_Float16, R / 8>(kl)) << 4) + ((col & 7) << 1);
            }
        }
    }
    // to the next slab: its own image lies `delta` bytes further, the one behind it `delta_next`
    __device__ __forceinline__ void move(int delta, int delta_next)
    {
#pragma unroll
        for (int x = 0; x < NA; ++x) at[x] += SKEW && KC && next[x] ? delta_next : delta;
    }
    __device__ __forceinline__ frag_t read(int f, int kg) const
    {
        if constexpr (KC) {
            return *(const GEMM_LDS(frag_t) *)(uintptr_t)(at[kg] + f * 32 * RBK);
        } else {
            const uint32_t p = at[f] + 16 * kg * (R * 2);
            const half4_t lo = __builtin_bit_cast(half4_t, __builtin_amdgcn_ds_read_tr16_b64_v4f16((GEMM_LDS(fp16x4_t) *)(uintptr_t)p));
            const half4_t hi = __builtin_bit_cast(half4_t, __builtin_amdgcn_ds_read_tr16_b64_v4f16((GEMM_LDS(fp16x4_t) *)(uintptr_t)(p + 4 * (R * 2))));
            return __builtin_bit_cast(frag_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        }
    }
};

// s_waitcnt vmcnt(slabs * NL) for slabs = min(left, MOST) (the count is an immediate)
template <int MOST, int NL> __device__ __forceinline__ void wait_slabs_left(int left)
{
    if constexpr (MOST > 0) {
        if (left < MOST) {
            wait_slabs_left<MOST - 1, NL>(left);
            return;
        }
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(MOST * NL));
}

template <typename T, int BM, int BN, int WM, int WN, int NST, bool AKC, bool BKC, bool SKEW>
__global__ __launch_bounds__(WM *WN * 64) void gemm_stage_kernel(const KernelArgs p)
{
    static_assert(sizeof(T) == 2, "16-bit operands");
    constexpr int NW = WM * WN;
    constexpr int BK = Elem<T>::BK, KG = Elem<T>::KG, EPC = Elem<T>::EPC;
    constexpr int TM = BM / WM, TN = BN / WN, FM = TM / 32, FN = TN / 32;
    constexpr int A_BYTES = BM * RBK, B_BYTES = BN * RBK, STAGE = A_BYTES + B_BYTES;
    typedef StageLoader<T, BM, NW, AKC, SKEW> LoaderA;
    typedef StageLoader<T, BN, NW, BKC, SKEW> LoaderB;
    constexpr int NVA = LoaderA::PER_WAVE, NVB = LoaderB::PER_WAVE, NL = NVA + NVB;  // loads per wave and slab
    static_assert(NST >= 3 + SKEW && (NST - 1) * NL <= 63, "the counted waits go up to 63 loads");
    constexpr int NB = FM * FN, NM = KGS * NB;  // MFMA blocks of a k-group and of a slab
    typedef typename Frag<T>::type frag_t;

    __shared__ __attribute__((aligned(1024))) char smem[NST * STAGE];
    GEMM_LDS(char) *lds = (GEMM_LDS(char) *)smem;
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int KT = (p.K + BK - 1) / BK;
    WorkItem item;
    if (!work_item(p, KT, item)) return;
    trace_mark(p, 0);
    trace_place<SKEW>(p);
    const int m0 = item.tile_m * BM, n0 = item.tile_n * BN;

    // slabs of this slice; only the operand's last one can be ragged
    const int kt0 = item.kt0, n = item.kt1 - kt0;
    const int krem = p.K - (kt0 + n - 1) * BK < BK ? p.K - (kt0 + n - 1) * BK : BK;  // k of the last slab
    const int images = n + SKEW;
    const bool safe = p.safe != 0;

    LoaderA la;
    LoaderB lb;
    la.init((const T *)p.A, p.lda, m0, p.M, p.K, kt0 * BK, wave, lane);
    lb.init((const T *)p.B, p.ldb, n0, p.N, p.K, kt0 * BK, wave, lane);
    const uint32_t dst_a = lds0 + wave * (NVA * 1024), dst_b = lds0 + A_BYTES + wave * (NVB * 1024);
    auto load1 = [&](int slot, int q) {  // load q of the loaders' slab into the slot at this LDS offset
        if (q < NVA) la.issue(dst_a + slot, q);
        else lb.issue(dst_b + slot, q - NVA);
    };
    int h = 0;  // slab (image) the loaders point at
    // Exact ranges from two slabs before the end on, because a granule of an M/N-contiguous operand with a leading
    // dimension below the granule covers up to four k-rows.
    auto prepare = [&]() {
        la.exact_range();
        lb.exact_range();
        if constexpr (SKEW) {
            const int left = krem - (h - (n - 1)) * BK;  // k from the image's beginning to the end of the last slab, none or less behind it
            if ((h == n - 1 && krem < BK) || h == n) {
                la.ragged_slab(left, wave, lane);
                lb.ragged_slab(left, wave, lane);
            }
            // the image behind the last slab is one of skewed rows only
            if (!AKC && h >= n) la.no_range();
            if (!BKC && h >= n) lb.no_range();
        } else if (h == n - 1 && krem < BK) {  // (apart from the above: the code that runs once costs by its length)
            la.ragged_slab(krem, wave, lane);
            lb.ragged_slab(krem, wave, lane);
        }
    };
    auto advance = [&]() {
        la.advance();
        lb.advance();
        if (++h >= n - 2) prepare();
    };
    // all but the youngest `left` slabs (MOST at most) landed; then the barrier
    auto hand_over = [&](auto most, int left) {
        if (safe) {
            full_sync();
        } else {
            wait_slabs_left<decltype(most)::value, NL>(left);
            barrier_keep_loads();
        }
    };
    typedef std::integral_constant<int, 1> One;
    typedef std::integral_constant<int, NST - 3 - SKEW> Ahead;
    auto load_first = [&](int slab) {
#pragma unroll
        for (int q = 0; q < NL; ++q) load1(slab * STAGE, q);
        advance();
    };
    if (n <= 2) prepare();
    load_first(0);
    if constexpr (SKEW) load_first(1);
    if (n > 1) load_first(1 + SKEW);

    float16_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    StageFragments<T, BM, AKC, FM, SKEW> ra;
    StageFragments<T, BN, BKC, FN, SKEW> rb;
    ra.init(lds0, wm * TM, lane, p.lda, p.M, STAGE);
    rb.init(lds0 + A_BYTES, wn * TN, lane, p.ldb, p.N, STAGE);
    frag_t fa[KGS][FM], fb[KGS][FN];
    auto read_group = [&](int kg) {
#pragma unroll
        for (int i = 0; i < FM; ++i) fa[kg][i] = ra.read(i, kg);
#pragma unroll
        for (int j = 0; j < FN; ++j) fb[kg][j] = rb.read(j, kg);
    };
    hand_over(One(), n - 1);  // slab 0 (and the image behind it: everything below speaks of slabs with theirs)
    trace_mark(p, 1);
#pragma unroll
    for (int kg = 0; kg < KGS; ++kg) {
        read_group(kg);
        __builtin_amdgcn_sched_barrier(0);  // the loop's waits count on this order
    }
#pragma unroll 1
    for (int i = 2 + SKEW; i < NST - 1 && i < images; ++i) load_first(i);
    hand_over(Ahead(), n - 2);  // slab 1

    // block m of a slab, k-group by k-group; blocks of a k-group in boustrophedon order, as in gemm_tile_kernel
    auto multiply1 = [&](int m) {
        const int kg = m / NB, b = m % NB;
        const int mi = b / FN, mj = (mi & 1) ? FN - 1 - b % FN : b % FN;
        mma(acc[mi][mj], fa[kg][mi], fb[kg][mj]);
        asm volatile("" : "+a"(acc[mi][mj]));  // keeps the MFMA at this place in the stream
    };
    int read_at = 0, free = (NST - 1) * STAGE;  // LDS offsets: of the slab in the fragment addresses, of the free slot
    // slab t, not the last one: multiply it, read slab t+1, load (if LOAD) slab (image) t+NST-1 into the free slot
    auto body = [&](auto load_tag, int left) {
        constexpr bool LOAD = decltype(load_tag)::value;
        const int delta = read_at == (NST - 1) * STAGE ? -(NST - 1) * STAGE : STAGE;
        const int delta_next = SKEW && read_at == (NST - 2) * STAGE ? -(NST - 1) * STAGE : STAGE;
        ra.move(delta, delta_next);
        rb.move(delta, delta_next);
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            multiply1(m);
            if (m % NB == NB - 1) read_group(m / NB);
            if constexpr (LOAD) {
#pragma unroll
                for (int q = 0; q < NL; ++q)
                    if (q * NM / NL == m) load1(free, q);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        free = read_at;
        read_at += delta;
        if constexpr (LOAD) advance();
        hand_over(Ahead(), left);  // slab t+2
    };
    int t = 0;
    for (; t + NST - 1 < images; ++t) body(std::true_type(), NST);
    for (; t < n - 1; ++t) body(std::false_type(), n - 3 - t);
    // the last slab
    if ((AKC || BKC) && krem % EPC != 0) {
        // elements past K in the granule that straddles it
        const int part = krem % EPC, half = krem % KG / EPC;
        uint4_t mask;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const int in = part * (int)sizeof(T) - 4 * w;  // bytes of this word inside K
            const uint32_t keep = in >= 4 ? 0xffffffffu : (in == 2 ? 0x0000ffffu : 0u);
            mask[w] = (lane >> 5) == half ? keep : 0xffffffffu;
        }
#pragma unroll
        for (int kg = 0; kg < KGS; ++kg) {
            if (kg != krem / KG) continue;
            if (AKC)
#pragma unroll
                for (int i = 0; i < FM; ++i) fa[kg][i] = __builtin_bit_cast(frag_t, __builtin_bit_cast(uint4_t, fa[kg][i]) & mask);
            if (BKC)
#pragma unroll
                for (int j = 0; j < FN; ++j) fb[kg][j] = __builtin_bit_cast(frag_t, __builtin_bit_cast(uint4_t, fb[kg][j]) & mask);
        }
    }
#pragma unroll
    for (int kg = 0; kg < KGS; ++kg) {
        if (kg * KG >= krem) break;
#pragma unroll
        for (int b = 0; b < NB; ++b) multiply1(kg * NB + b);
    }
    trace_mark(p, 2);
    store_tile<BM, BN, WM, WN, NST * STAGE>(p, item, acc, lds, m0, n0, wave, lane);
}

}  // namespace gemm_gfx950
