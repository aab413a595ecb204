// Binary32 products on the bfloat16 matrix instructions.
//
// v_mfma_f32_32x32x2_f32 runs at a sixteenth of the bfloat16 rate, so a binary32 product is bound by
// the matrix cores.  Here every binary32 operand is written as the sum of three
// bfloat16 numbers, x = h + m + l (each the rounding to nearest of what the ones before leave: 3 x 8
// significant bits hold the 24 of x exactly), and the six products that reach down to 2^-18 of the
// largest, hh + hm + mh + mm + hl + lh, are accumulated in binary32.  What is left out, ml + lm + ll, is
// below 2^-25 of |x y| with random sign: less than the rounding of one binary32 addition.  One
// 32x32x16 block takes 6 matrix instructions of 32 cycles instead of 8 of 64.
//
// The split is exact unless an operand has bits below 2^-133, which bfloat16 subnormals do not
// reach (|x| below about 2^-110); NaN, infinity and values that round to infinity leave a non-finite
// accumulator.  A workgroup in whose operands or results either was seen computes its tile
// again with the binary32 matrix instructions (exact_tile), so every input gives what those give.
//
// Operands go global -> registers -> (split) -> LDS, each element split once per workgroup.
// LDS image of one operand for one step of SK k: three planes (h, m, l), each laid out as the 16-bit
// images of the tile kernel: K-contiguous operand [tile row][SK], M/N-contiguous operand
// [k][R].  Tiles with few blocks per wave keep three buffers, the others two (see AHEAD); while a step is multiplied,
// registers that hold a later one are split, written to a free buffer and refilled; one barrier per step.
// What bounds it: power at 4096^3 (matrix cores busy 75 % of the time at 1.8 GHz; 912 us on the binary32 instructions,
// 577 here); one workgroup per CU at 2048^3 (128 -> 94 us), where loads, splitting and hand-over show.
// Nothing writes LDS behind the program's back here (no direct loads), so every hand-over is fully
// synchronised and KernelArgs::safe changes nothing.
#pragma once
#include "gemm_kernel.h"

namespace gemm_gfx950 {

typedef float float2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t uint2_t __attribute__((ext_vector_type(2)));

// Sums shorter than this are left to the binary32 instructions: these round once per product and the split's six
// products up to six times per k-group, so below two k-groups they are the more exact (error against binary64 of a
// 512x512xK product, 2-norm, binary32 instructions / split: K = 1 2.5e-8 / 5.2e-8, 16 7.3e-8 / 8.2e-8, 32 1.03e-7 /
// 1.04e-7, 64 1.44e-7 / 1.35e-7, 512 4.1e-7 / 3.5e-7, 32768 3.2e-6 / 3.0e-6).
constexpr int kSplitMinK = 64;
constexpr int kSplitMaxK = 2048;  // terms per accumulator the selection does not exceed in long sums (error 7e-7 there)

// Two operands as three pairs of bfloat16; rest collects the bits the three pieces do not hold
// (bits 0..15 nonzero: the split was not exact).
__device__ __forceinline__ void split_pair(float x0, float x1, uint32_t &h, uint32_t &m, uint32_t &l, uint32_t &rest)
{
    h = __builtin_bit_cast(uint32_t, __builtin_convertvector((float2_t){x0, x1}, bf16x2_t));
    const float r0 = x0 - __builtin_bit_cast(float, h << 16);
    const float r1 = x1 - __builtin_bit_cast(float, h & 0xffff0000u);
    m = __builtin_bit_cast(uint32_t, __builtin_convertvector((float2_t){r0, r1}, bf16x2_t));
    const uint32_t q0 = __builtin_bit_cast(uint32_t, r0 - __builtin_bit_cast(float, m << 16));
    const uint32_t q1 = __builtin_bit_cast(uint32_t, r1 - __builtin_bit_cast(float, m & 0xffff0000u));
    l = __builtin_amdgcn_perm(q1, q0, 0x07060302);  // the upper halves; the lower ones are zero if the split is exact
    rest |= q0 | q1;
}

// Loader of one operand, R tile rows by SK k per step.  A thread owns PER quads of four consecutive
// elements of the contiguous dimension; consecutive lanes own consecutive quads, so a load
// instruction covers whole rows of the slab.
template <int R, int NT, int SK, bool KC>
struct SplitLoader {
    static constexpr int QUADS = R * SK / 4, PER = QUADS / NT;
    static_assert(QUADS % NT == 0 && PER >= 1, "tile too small for this workgroup");
    static constexpr int GPS = SK / 8;               // 16-byte granules per row of a K-contiguous plane
    static constexpr int PLANE = R * SK * 2;         // bytes
    static constexpr int BYTES = 3 * PLANE;
    typedef float quad_t __attribute__((ext_vector_type(4), aligned(4)));

    const char *base;      // uniform: first k of the next step to load
    int64_t step;          // bytes per step
    uint32_t off[PER];     // this thread's quads relative to base

    static __device__ __forceinline__ void place(int q, int &row, int &k)
    {
        if (KC) { row = q / (SK / 4); k = 4 * (q % (SK / 4)); }
        else { k = q / (R / 4); row = 4 * (q % (R / 4)); }
    }
    __device__ __forceinline__ void init(const float *origin, int64_t ld, int row0, int rmax, int k0, int tid)
    {
        base = (const char *)(KC ? origin + (int64_t)row0 * ld + k0 : origin + (int64_t)k0 * ld + row0);
        step = (KC ? (int64_t)SK : (int64_t)SK * ld) * 4;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            int row, k;
            place(tid + i * NT, row, k);
            if (KC) row = row0 + row < rmax ? row : rmax - 1 - row0;  // rows past the edge re-read the last one
            else row = row0 + row < rmax ? row : 0;                   // quads past the edge re-read the first one
            off[i] = (uint32_t)((KC ? (int64_t)row * ld + k : (int64_t)k * ld + row) * 4);
        }
    }
    __device__ __forceinline__ float4_t load1(int i) const { return *(const quad_t *)(base + off[i]); }
    __device__ __forceinline__ void advance() { base += step; }
    __device__ __forceinline__ void load(float4_t (&v)[PER])
    {
#pragma unroll
        for (int i = 0; i < PER; ++i) v[i] = load1(i);
        advance();
    }
    // the step that starts at k, whatever part of it lies inside the matrix and below kend; zero outside
    static __device__ __forceinline__ void load_guarded(float4_t (&v)[PER], const float *origin, int64_t ld, int row0,
                                                        int rmax, int k0, int kend, int tid)
    {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            int row, k;
            place(tid + i * NT, row, k);
            row += row0;
            k += k0;
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const bool in = KC ? (row < rmax && k + x < kend) : (row + x < rmax && k < kend);
                const float *p = KC ? origin + (int64_t)row * ld + k + x : origin + (int64_t)k * ld + row + x;
                v[i][x] = in ? *p : 0.0f;
            }
        }
    }
    static __device__ __forceinline__ int slot_of(int q)  // byte position of quad q inside a plane
    {
        int row, k;
        place(q, row, k);
        if (KC) {
            const int g = (k >> 3) ^ ((row / (16 / GPS)) & (GPS - 1));
            return row * (SK * 2) + (g << 4) + ((k & 4) << 1);
        }
        return k * (R * 2) + (((row >> 3) ^ swz_mc<_Float16, R / 8>(k)) << 4) + ((row & 4) << 1);
    }
    // one half (two elements) of quad i split into its pieces; the second half also writes the quad to LDS
    template <int HALF>
    static __device__ __forceinline__ void split(GEMM_LDS(char) *img, int tid, int i, const float4_t &v, uint2_t (&piece)[3],
                                                 uint32_t &rest)
    {
        uint32_t a, b, c;
        split_pair(v[2 * HALF], v[2 * HALF + 1], a, b, c, rest);
        piece[0][HALF] = a;
        piece[1][HALF] = b;
        piece[2][HALF] = c;
        if constexpr (HALF == 1) {
            GEMM_LDS(char) *d = img + slot_of(tid + i * NT);
#pragma unroll
            for (int x = 0; x < 3; ++x) *(GEMM_LDS(uint2_t) *)(d + x * PLANE) = piece[x];
        }
    }
    // operand of one 32x32x16 instruction: rows r0.., k-group kg of the step, one plane
    static __device__ __forceinline__ bf16x8_t fetch(const GEMM_LDS(char) *plane, int r0, int kg, int lane)
    {
        if constexpr (KC) {
            const int r = r0 + (lane & 31);
            const int g = (2 * kg + (lane >> 5)) ^ ((r / (16 / GPS)) & (GPS - 1));
            return *(const GEMM_LDS(bf16x8_t) *)(plane + r * (SK * 2) + (g << 4));
        } else {
            // 16 k-rows further on the swizzle is the same
            return __builtin_bit_cast(bf16x8_t, fetch_f16_mc_kg<R, 0>(plane + kg * 16 * (R * 2), r0, lane));
        }
    }
};

// The tile with the binary32 matrix instructions, any operands: guarded loads through one pair of LDS buffers.
template <int BM, int BN, int WM, int WN, bool AKC, bool BKC>
__device__ __forceinline__ void exact_tile(const KernelArgs &p, float16_t (&acc)[BM / WM / 32][BN / WN / 32],
                                           GEMM_LDS(char) *lds, int m0, int n0, int k0, int kend, int wave, int lane, int tid,
                                           bool active)
{
    constexpr int NT = WM * WN * 64, TM = BM / WM, TN = BN / WN, FM = TM / 32, FN = TN / 32, BK = Elem<float>::BK;
    const int wm = wave / WN, wn = wave % WN;
    const float *A = (const float *)p.A, *B = (const float *)p.B;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    GEMM_LDS(char) *iA = lds, *iB = lds + BM * RBK;
    for (int k = k0; k < kend; k += BK) {
        __syncthreads();
        if (active) {
            Staged<float, BM, NT> sa;
            guarded_fetch<float, BM, NT, AKC>(sa, A, p.lda, m0, p.M, k, kend, tid);
            staged_store<float, BM, NT, AKC>(iA, sa, A, p.lda, m0, p.M, k, kend, tid);
        }
        if (active) {
            Staged<float, BN, NT> sb;
            guarded_fetch<float, BN, NT, BKC>(sb, B, p.ldb, n0, p.N, k, kend, tid);
            staged_store<float, BN, NT, BKC>(iB, sb, B, p.ldb, n0, p.N, k, kend, tid);
        }
        __syncthreads();
#pragma unroll 1
        for (int kg = 0; kg < KGS; ++kg) {
            float4_t fa[FM], fb[FN];
#pragma unroll
            for (int i = 0; i < FM; ++i) fa[i] = Fetch<float, BM, AKC>::get(iA, wm * TM + i * 32, kg, lane);
#pragma unroll
            for (int j = 0; j < FN; ++j) fb[j] = Fetch<float, BN, BKC>::get(iB, wn * TN + j * 32, kg, lane);
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) mma(acc[i][j], fa[i], fb[j]);
        }
    }
}

// Waves of a workgroup: WM x WN over the tile, times WK over k (each of the WK groups multiplies one k-group of
// every step; their accumulators are added at the end).  With several groups a lone workgroup keeps more than
// one wave per SIMD, whose fetches, splitting and matrix instructions fill each other's gaps.
constexpr int f32_wave_groups(int BM, int BN) { return BM == 128 && BN == 128 ? 2 : 1; }
constexpr int f32_waves_per_simd(int BM, int BN, int NW) { return BM * BN <= 128 * 128 || NW == 8 ? 2 : 1; }

template <int BM, int BN, int WM, int WN, bool AKC, bool BKC>
__global__ __launch_bounds__(WM *WN *f32_wave_groups(BM, BN) * 64, f32_waves_per_simd(BM, BN, WM * WN)) void gemm_f32_kernel(const KernelArgs p)
{
    constexpr int WK = f32_wave_groups(BM, BN);
    constexpr int NW = WM * WN, NT = NW * WK * 64;
    constexpr int BK = Elem<float>::BK;
    constexpr int TM = BM / WM, TN = BN / WN, FM = TM / 32, FN = TN / 32, NB = FM * FN;
    constexpr int SK = 16 * WK;                            // k per step: one k-group per wave
    // Waves with few blocks finish a product before the next one's pieces could be fetched.  They have three LDS
    // buffers: while step s is multiplied from registers, all pieces of step s+1 are fetched and step s+2 is split.
    constexpr bool AHEAD = NB < 8;
    constexpr int NBUF = AHEAD ? 3 : 2, LOOK = NBUF - 1;   // step s splits step s + LOOK
    constexpr int DEPTH = AHEAD ? (WK == 2 ? 1 : 3) : (BM * BN < 256 * 256 ? 2 : 1);  // steps in flight in registers
    constexpr int UNROLL = NBUF;                           // steps after which buffers and register sets repeat
    static_assert(UNROLL % DEPTH == 0, "register sets repeat with the buffers");
    constexpr int BARRIER_Q = AHEAD ? 6 : 5;               // the product the barrier stands before (6: after the last)
    typedef SplitLoader<BM, NT, SK, AKC> LA;
    typedef SplitLoader<BN, NT, SK, BKC> LB;
    constexpr int BUF = LA::BYTES + LB::BYTES;
    constexpr int EXACT = (BM + BN) * RBK;                 // LDS of exact_tile
    constexpr int LDS_BYTES = NBUF * BUF > EXACT ? NBUF * BUF : EXACT;

    __shared__ __attribute__((aligned(1024))) char smem[LDS_BYTES];
    GEMM_LDS(char) *lds = (GEMM_LDS(char) *)smem;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave_id = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int group = wave_id / NW, wave = wave_id % NW;
    const int wm = wave / WN, wn = wave % WN;

    // same work-item order as gemm_tile_kernel: one contiguous run per XCD, K-slice by K-slice
    const int ntiles = p.tiles_m * p.tiles_n;
    const int nwork = ntiles * p.splits;
    const int per_xcd = (nwork + 7) >> 3;
    const int work = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (work >= nwork) return;
    trace_mark(p, 0);
    trace_place(p);
    const int slice = work / ntiles;
    const int lin = work - slice * ntiles;
    constexpr int GM = 8;
    const int band = lin / (GM * p.tiles_n);
    const int first_m = band * GM;
    const int band_rows = (p.tiles_m - first_m) < GM ? (p.tiles_m - first_m) : GM;
    const int in_band = lin - band * GM * p.tiles_n;
    const int tile_m = first_m + in_band % band_rows;
    const int tile_n = in_band / band_rows;
    const int m0 = tile_m * BM, n0 = tile_n * BN;

    const int k0 = slice * p.kt_per_split * BK;
    const int64_t kend_slice = (int64_t)(slice + 1) * p.kt_per_split * BK;
    const int kend = kend_slice < p.K ? (int)kend_slice : p.K;

    const float *A = (const float *)p.A, *B = (const float *)p.B;

    float16_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    // Steps 0 .. nfast-1 are loaded with whole quads.  A quad of an M/N-contiguous operand that straddles the matrix
    // edge is read whole (its tail only feeds results that are never stored); on the operand's last k-row that tail
    // could lie past the operand, so a tile with such quads loads the last step guarded, like the rest of a ragged K.
    const bool edge_a = !AKC && (p.M & 3) != 0 && m0 + BM > p.M;
    const bool edge_b = !BKC && (p.N & 3) != 0 && n0 + BN > p.N;
    const bool split = p.K >= kSplitMinK;
    const int n = split ? (kend - k0 + SK - 1) / SK : 0;
    int nfast = split ? (kend - k0) / SK : 0;
    if ((edge_a || edge_b) && k0 + nfast * SK == p.K) --nfast;
    if (!p.ld32 || (edge_a && p.lda < 8) || (edge_b && p.ldb < 8)) nfast = 0;

    LA la;
    LB lb;
    la.init(A, p.lda, m0, p.M, k0, tid);
    lb.init(B, p.ldb, n0, p.N, k0, tid);
    float4_t ra[DEPTH][LA::PER], rb[DEPTH][LB::PER];  // step s waits in set s % DEPTH
    uint32_t rest = 0;

    // loads of any step (uniform branch)
    auto load_any = [&](auto set_tag, int s) {
        constexpr int S = decltype(set_tag)::value;
        if (s < nfast) {
            la.load(ra[S]);
            lb.load(rb[S]);
        } else if (s < n) {
            LA::load_guarded(ra[S], A, p.lda, m0, p.M, k0 + s * SK, kend, tid);
            LB::load_guarded(rb[S], B, p.ldb, n0, p.N, k0 + s * SK, kend, tid);
        }
    };
    // half u & 1 of quad u / 2 of the set; then, if `refill`, the load that refills the quad
    uint2_t piece[3];
    auto split_unit = [&](auto set_tag, int u, GEMM_LDS(char) *buf, bool refill) {
        constexpr int S = decltype(set_tag)::value;
        const int q = u >> 1;
        if (q < LA::PER) {
            if ((u & 1) == 0) LA::template split<0>(buf, tid, q, ra[S][q], piece, rest);
            else LA::template split<1>(buf, tid, q, ra[S][q], piece, rest);
            if ((u & 1) && refill) ra[S][q] = la.load1(q);
        } else {
            if ((u & 1) == 0) LB::template split<0>(buf + LA::BYTES, tid, q - LA::PER, rb[S][q - LA::PER], piece, rest);
            else LB::template split<1>(buf + LA::BYTES, tid, q - LA::PER, rb[S][q - LA::PER], piece, rest);
            if ((u & 1) && refill) rb[S][q - LA::PER] = lb.load1(q - LA::PER);
        }
    };
    constexpr int UNITS = 2 * (LA::PER + LB::PER);
    auto hand_over = [&]() {
        __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(63));  // own LDS reads and writes done; global loads stay in flight
        barrier_keep_loads();
    };
    // operands of this wave's k-group of a step: piece x, block row i / block column j
    auto fetch_a = [&](const GEMM_LDS(char) *buf, int x, int i) {
        return LA::fetch(buf + x * LA::PLANE, wm * TM + i * 32, group, lane);
    };
    auto fetch_b = [&](const GEMM_LDS(char) *buf, int x, int j) {
        return LB::fetch(buf + LA::BYTES + x * LB::PLANE, wn * TN + j * 32, group, lane);
    };
    typedef std::integral_constant<int, 0> I0;
    typedef std::integral_constant<int, 1> I1;
    typedef std::integral_constant<int, 2> I2;

#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
#pragma unroll
        for (int i = 0; i < LA::PER; ++i) ra[d][i] = 0.0f;
#pragma unroll
        for (int i = 0; i < LB::PER; ++i) rb[d][i] = 0.0f;
    }
    load_any(I0(), 0);
    if constexpr (DEPTH > 1) load_any(std::integral_constant<int, 1 % DEPTH>(), 1);
    if constexpr (DEPTH > 2) load_any(std::integral_constant<int, 2 % DEPTH>(), 2);
    static_assert(DEPTH <= 3, "prologue written for up to three register sets");
#pragma unroll
    for (int u = 0; u < UNITS; ++u) split_unit(I0(), u, lds, false);
    load_any(I0(), DEPTH);
    if constexpr (LOOK == 2) {
#pragma unroll
        for (int u = 0; u < UNITS; ++u) split_unit(std::integral_constant<int, 1 % DEPTH>(), u, lds + BUF, false);
        load_any(std::integral_constant<int, 1 % DEPTH>(), 1 + DEPTH);
    }
    hand_over();
    trace_mark(p, 1);

    // pieces of the k-group to multiply next: all of them (AHEAD), or the h pieces only
    constexpr int NX = AHEAD ? 3 : 1;
    bf16x8_t fa[NX][FM], fb[NX][FN];
#pragma unroll
    for (int x = 0; x < NX; ++x) {
#pragma unroll
        for (int i = 0; i < FM; ++i) fa[x][i] = fetch_a(lds, x, i);
#pragma unroll
        for (int j = 0; j < FN; ++j) fb[x][j] = fetch_b(lds, x, j);
    }

    int s = 0;
    // Multiplies step s (a multiple of UNROLL plus D), splits step s+LOOK into its LDS buffer and refills its registers
    // with step s+LOOK+DEPTH, in a fixed order (the compiler may not move anything across the fences): the six products one
    // after the other, and between their matrix instructions the fetches of pieces needed later and
    // the splitting, so that vector and LDS work runs in the shadow of the matrix cores.
    auto body = [&](auto d_tag, auto fast_tag) {
        constexpr bool FAST = decltype(fast_tag)::value;
        constexpr int D = decltype(d_tag)::value;
        std::integral_constant<int, (D + LOOK) % DEPTH> set;
        constexpr int SPAN = (AHEAD ? 5 : BARRIER_Q) * NB;  // matrix instructions the splitting is spread over
        GEMM_LDS(char) *now = lds + (D % NBUF) * BUF, *next = lds + ((D + 1) % NBUF) * BUF;
        GEMM_LDS(char) *fill = lds + ((D + LOOK) % NBUF) * BUF;
        bf16x8_t am[FM], al[FM], bm[FN], bl[FN];  // !AHEAD: fetched one product early
        bf16x8_t na[NX][FM], nb[NX][FN];          // for the next step
        if constexpr (AHEAD) {
#pragma unroll
            for (int i = 0; i < FM; ++i) { am[i] = fa[NX / 2][i]; al[i] = fa[NX - 1][i]; }
#pragma unroll
            for (int j = 0; j < FN; ++j) { bm[j] = fb[NX / 2][j]; bl[j] = fb[NX - 1][j]; }
        }
        constexpr int FQ = AHEAD ? 0 : 5;                                // product the fetches of the next step begin at
        constexpr int NFN = NX * (FM + FN), FSPAN = AHEAD ? 4 * NB : NB;  // their number, and the instructions they are spread over
        auto product = [&](auto q_tag, const bf16x8_t(&a)[FM], const bf16x8_t(&b)[FN]) {
            constexpr int Q = decltype(q_tag)::value;
            if constexpr (Q == 5 && !FAST) load_any(set, s + LOOK + DEPTH);
            if constexpr (Q == BARRIER_Q) hand_over();
#pragma unroll
            for (int m = 0; m < NB; ++m) {
                const int i = m / FN, j = (i & 1) ? FN - 1 - m % FN : m % FN;
                mma(acc[i][j], a[i], b[j]);
                // An ordered use of the result keeps the matrix instruction at this place.  Accumulation registers where a
                // wave owns the SIMD's 512; with several waves per SIMD the compiler would halve each wave's
                // share between the two kinds, so there the accumulators stay in ordinary registers.
                if constexpr (f32_waves_per_simd(BM, BN, WM * WN) == 1) asm volatile("" : "+a"(acc[i][j]));
                else asm volatile("" : "+v"(acc[i][j]));
                if constexpr (!AHEAD) {
                    constexpr int NF = Q < 2 ? FN : (Q < 4 ? FM : 0);
#pragma unroll
                    for (int f = 0; f < NF; ++f) {
                        if ((f < NB ? f : NB - 1) != m) continue;
                        if (Q == 0) bm[f] = fetch_b(now, 1, f);
                        if (Q == 1) bl[f] = fetch_b(now, 2, f);
                        if (Q == 2) am[f] = fetch_a(now, 1, f);
                        if (Q == 3) al[f] = fetch_a(now, 2, f);
                    }
                }
                if constexpr (Q >= FQ) {
#pragma unroll
                    for (int f = 0; f < NFN; ++f) {
                        if (f * FSPAN / NFN != (Q - FQ) * NB + m) continue;
                        const int x = f / (FM + FN), y = f % (FM + FN);
                        if (y < FM) na[x][y] = fetch_a(next, x, y);
                        else nb[x][y - FM] = fetch_b(next, x, y - FM);
                    }
                }
#pragma unroll
                for (int u = 0; u < UNITS; ++u)
                    if (u * SPAN / UNITS == Q * NB + m) split_unit(set, u, fill, FAST);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        product(std::integral_constant<int, 0>(), fa[0], fb[0]);
        product(std::integral_constant<int, 1>(), fa[0], bm);
        product(std::integral_constant<int, 2>(), fa[0], bl);
        product(std::integral_constant<int, 3>(), am, bm);
        product(std::integral_constant<int, 4>(), am, fb[0]);
        product(std::integral_constant<int, 5>(), al, fb[0]);
        if constexpr (BARRIER_Q == 6) hand_over();
#pragma unroll
        for (int x = 0; x < NX; ++x) {
#pragma unroll
            for (int i = 0; i < FM; ++i) fa[x][i] = na[x][i];
#pragma unroll
            for (int j = 0; j < FN; ++j) fb[x][j] = nb[x][j];
        }
        if constexpr (FAST) {
            la.advance();
            lb.advance();
        }
        ++s;
    };
    // whole rounds in which every load is one of whole quads
    while (s + UNROLL - 1 + LOOK + DEPTH < nfast) {
        body(I0(), std::true_type());
        body(I1(), std::true_type());
        if constexpr (UNROLL > 2) body(I2(), std::true_type());
    }
    // the last steps: nothing, or only part of a step, is left to load
    while (s < n) {
        body(I0(), std::false_type());
        if (s < n) body(I1(), std::false_type());
        if constexpr (UNROLL > 2) { if (s < n) body(I2(), std::false_type()); }
    }

    // the groups' sums, added by the first
    if constexpr (WK > 1) {
        constexpr int PART = NB * 16 * NW * 64;  // floats of one group
        static_assert((WK - 1) * PART * 4 <= LDS_BYTES, "the accumulators fit the operand buffers");
        GEMM_LDS(float) *part = (GEMM_LDS(float) *)lds + (wave * 64 + lane);
        __syncthreads();  // the operand buffers have been read
#pragma unroll
        for (int x = 0; x < NB * 16; ++x)
            if (group > 0) part[(group - 1) * PART + x * (NW * 64)] = acc[x / 16 / FN][x / 16 % FN][x % 16];
        __syncthreads();
        if (group == 0) {
#pragma unroll
            for (int x = 0; x < NB * 16; ++x)
#pragma unroll
                for (int g = 0; g < WK - 1; ++g) acc[x / 16 / FN][x / 16 % FN][x % 16] += part[g * PART + x * (NW * 64)];
        }
    }

    // anything the split does not serve: not all bits held, or a result inside C that is no number
    bool bad = !split || (rest & 0xffffu) != 0;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            uint32_t top = 0;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const bool in = m0 + wm * TM + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3) < p.M;
                const uint32_t e = __builtin_bit_cast(uint32_t, (float)acc[i][j][r]) & 0x7fffffffu;
                top = in && e > top ? e : top;
            }
            bad = bad || (group == 0 && top >= 0x7f800000u && n0 + wn * TN + j * 32 + (lane & 31) < p.N);
        }
    if (__syncthreads_or(bad))
        exact_tile<BM, BN, WM, WN, AKC, BKC>(p, acc, lds, m0, n0, k0, kend, wave, lane, tid, group == 0);

    trace_mark(p, 2);
    store_tile<BM, BN, WM, WN, LDS_BYTES>(p, acc, lds, slice, m0, n0, wave, lane, group == 0);
}

}  // namespace gemm_gfx950
