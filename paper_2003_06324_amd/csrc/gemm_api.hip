// C ABI of the library: argument validation, per-shape tile / split-K
// selection (the paper picks the block tile per input size, Section 5.3), and
// kernel launches on the caller's stream.  No host synchronisation.
#include "gemm.h"
#include "gemm_launch.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <tuple>
#include <type_traits>
#include <utility>
#include <vector>

using namespace gemm_gfx950;

namespace gemm_gfx950 {
GEMM_DECLARE_TILE(_Float16, 256, 256, 2, 2)
GEMM_DECLARE_TILE(_Float16, 256, 256, 2, 4)
GEMM_DECLARE_TILE(_Float16, 128, 128, 2, 2)
GEMM_DECLARE_TILE(_Float16, 64, 64, 2, 2)
GEMM_DECLARE_TILE(_Float16, 256, 128, 2, 2)
GEMM_DECLARE_TILE(_Float16, 128, 256, 2, 2)
GEMM_DECLARE_TILE(_Float16, 128, 64, 2, 2)
GEMM_DECLARE_TILE(_Float16, 64, 128, 2, 2)
GEMM_DECLARE_TILE(__bf16, 256, 256, 2, 2)
GEMM_DECLARE_TILE(__bf16, 256, 256, 2, 4)
GEMM_DECLARE_TILE(__bf16, 128, 128, 2, 2)
GEMM_DECLARE_TILE(__bf16, 64, 64, 2, 2)
GEMM_DECLARE_TILE(__bf16, 256, 128, 2, 2)
GEMM_DECLARE_TILE(__bf16, 128, 256, 2, 2)
GEMM_DECLARE_TILE(__bf16, 128, 64, 2, 2)
GEMM_DECLARE_TILE(__bf16, 64, 128, 2, 2)
GEMM_DECLARE_TILE(float, 256, 256, 2, 2)
GEMM_DECLARE_TILE(float, 256, 256, 2, 4)
GEMM_DECLARE_TILE(float, 128, 128, 2, 2)
GEMM_DECLARE_TILE(float, 64, 64, 2, 2)
GEMM_DECLARE_TILE(float, 256, 128, 2, 2)
GEMM_DECLARE_TILE(float, 128, 256, 2, 2)
GEMM_DECLARE_TILE(float, 128, 64, 2, 2)
GEMM_DECLARE_TILE(float, 64, 128, 2, 2)
GEMM_DECLARE_KSPLIT(_Float16, 64, 64)
GEMM_DECLARE_KSPLIT(__bf16, 64, 64)
GEMM_DECLARE_KSPLIT(float, 64, 64)
GEMM_DECLARE_STAGE(_Float16, 64, 64, 6)
GEMM_DECLARE_STAGE(_Float16, 64, 128, 5)
GEMM_DECLARE_STAGE(_Float16, 128, 64, 5)
GEMM_DECLARE_STAGE(_Float16, 128, 128, 4)
GEMM_DECLARE_SKEW(_Float16, 64, 64, 7)
GEMM_DECLARE_SKEW(_Float16, 64, 128, 6)
GEMM_DECLARE_SKEW(_Float16, 128, 64, 6)
GEMM_DECLARE_SKEW(_Float16, 128, 128, 5)
GEMM_DECLARE_STAGE(__bf16, 64, 64, 6)
GEMM_DECLARE_STAGE(__bf16, 64, 128, 5)
GEMM_DECLARE_STAGE(__bf16, 128, 64, 5)
GEMM_DECLARE_STAGE(__bf16, 128, 128, 4)
GEMM_DECLARE_SKEW(__bf16, 64, 64, 7)
GEMM_DECLARE_SKEW(__bf16, 64, 128, 6)
GEMM_DECLARE_SKEW(__bf16, 128, 64, 6)
GEMM_DECLARE_SKEW(__bf16, 128, 128, 5)
GEMM_DECLARE_SMALL(_Float16)
GEMM_DECLARE_SMALL(__bf16)
GEMM_DECLARE_SMALL(float)
extern template hipError_t launch_small16<float>(bool, bool, dim3, hipStream_t, const KernelArgs &);
}  // namespace gemm_gfx950

namespace {

// Sums the K-slices of the workspace in slice order (deterministic) into C; TC is float, or
// _Float16 for the binary16-output entry point (one rounding, to nearest even, of the sum).
// A workspace row holds ldw floats, a multiple of 32 (ws_pitch): whatever N is, a thread takes
// four neighbouring columns with 16-byte loads, and rows begin on cache-line boundaries.  The
// loads of four slices are issued together and then added one after the other, in slice order:
// the pass is bound by memory latency, not by the additions.  vec_c: base and rows of C allow
// one store of the four results.
template <typename TC>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float *ws, int64_t split_stride,
                                                            int splits, int ldw, TC *C, int64_t ldc,
                                                            int M, int N, int vec_c)
{
    typedef float vec_t __attribute__((ext_vector_type(4)));
    typedef TC out_t __attribute__((ext_vector_type(4)));
    const int pieces = (N + 3) / 4;  // 16-byte pieces of a row that hold results
    const int64_t total = (int64_t)M * pieces;
    for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * 256) {
        const int64_t r = idx / pieces;
        const int c = (int)(idx - r * pieces) * 4;
        const float *src = ws + r * ldw + c;
        vec_t s = 0.0f;
        int z = 0;
        for (; z + 4 <= splits; z += 4) {
            const vec_t v0 = *(const vec_t *)(src + (z + 0) * split_stride);
            const vec_t v1 = *(const vec_t *)(src + (z + 1) * split_stride);
            const vec_t v2 = *(const vec_t *)(src + (z + 2) * split_stride);
            const vec_t v3 = *(const vec_t *)(src + (z + 3) * split_stride);
            s += v0;
            s += v1;
            s += v2;
            s += v3;
        }
        for (; z < splits; ++z) s += *(const vec_t *)(src + z * split_stride);
        TC *dst = C + r * ldc + c;
        if (vec_c && c + 4 <= N) {
            out_t o;
#pragma unroll
            for (int x = 0; x < 4; ++x) o[x] = (TC)s[x];
            *(out_t *)dst = o;
        } else {
            // (the columns of the last piece beyond N were never written by the product kernel
            // and are not stored)
#pragma unroll
            for (int x = 0; x < 4; ++x)
                if (c + x < N) dst[x] = (TC)s[x];
        }
    }
}

// Sums the partial tiles of a launch whose last tiles were sliced (KernelArgs::whole_tiles) in slice order into C: the
// same pass over packed tiles, [slice][tile][BM][BN].  grid.y: tile; the pieces of a tile (four columns) are shared out in x.
template <typename TC>
__global__ __launch_bounds__(256) void tail_reduce_kernel(const float *ws, int splits, int whole_tiles, int tiles_m, int tiles_n,
                                                          Divisor by_band, Divisor by_last_rows, int BM, int BN, TC *C, int64_t ldc, int M, int N, int vec_c)
{
    typedef float vec_t __attribute__((ext_vector_type(4)));
    typedef TC out_t __attribute__((ext_vector_type(4)));
    int tile_m, tile_n;
    tile_at(tiles_m, tiles_n, by_band, by_last_rows, whole_tiles + blockIdx.y, tile_m, tile_n);
    const int idx = (blockIdx.x * 256 + threadIdx.x) * 4;  // element of the tile; the grid holds exactly BM * BN / 4 threads a tile
    const int row = tile_m * BM + idx / BN, col = tile_n * BN + idx % BN;
    if (row >= M || col >= N) return;
    const int64_t stride = (int64_t)(tiles_m * tiles_n - whole_tiles) * BM * BN;
    const float *src = ws + (int64_t)blockIdx.y * BM * BN + idx;
    vec_t s = 0.0f;
    int z = 0;
    for (; z + 4 <= splits; z += 4) {
        const vec_t v0 = *(const vec_t *)(src + (z + 0) * stride);
        const vec_t v1 = *(const vec_t *)(src + (z + 1) * stride);
        const vec_t v2 = *(const vec_t *)(src + (z + 2) * stride);
        const vec_t v3 = *(const vec_t *)(src + (z + 3) * stride);
        s += v0;
        s += v1;
        s += v2;
        s += v3;
    }
    for (; z < splits; ++z) s += *(const vec_t *)(src + z * stride);
    TC *dst = C + (int64_t)row * ldc + col;
    if (vec_c && col + 4 <= N) {
        out_t o;
#pragma unroll
        for (int x = 0; x < 4; ++x) o[x] = (TC)s[x];
        *(out_t *)dst = o;
    } else {
#pragma unroll
        for (int x = 0; x < 4; ++x)
            if (col + x < N) dst[x] = (TC)s[x];
    }
}

template <typename TC>
__global__ __launch_bounds__(256) void fill_zero_kernel(TC *C, int64_t ldc, int M, int N)
{
    const int64_t total = (int64_t)M * N;
    for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * 256) {
        const int64_t r = idx / N, c = idx - r * N;
        C[r * ldc + c] = (TC)0.0f;
    }
}

constexpr int kDefaultNumCU = 256;  // MI355X; the launch path asks the device (gemm_query_config uses this)

// Partial results of the entry points that may not allocate (gemm_*_noalloc): one fixed array
// per GPU, held until the process ends.  Host code never passes this name to a kernel: it is a
// host-side stand-in; the device address comes from hipGetSymbolAddress (static_scratch()).
static __device__ __align__(256) unsigned char scratch[GEMM_NOALLOC_SCRATCH_BYTES];

struct TileConfig {
    const char *name;
    int BM, BN;
    int wg_per_cu;              // resident workgroups per CU (LDS-limited)
    double f16_alone, f16_full; // microseconds per 64-k slab: one workgroup on a CU / CU fully occupied
    double f32_alone, f32_full; // same per 32-k f32 slab
    double fixed;               // microseconds a round of tiles spends outside its K loop (first operands, stores)
    double hbm_eff;             // share of the model's HBM rate this tile's access pattern reaches
    double f16_a4, f32_a4;      // slab time on 4-/8-byte aligned operands (direct loads whose row pieces straddle
                                // cache lines) over the aligned slab time
    double f16_a2;              // same for 2-byte aligned 16-bit operands (register-staged, every 16-byte load split up)
    double general;             // same for the register-staged path on aligned 16-bit operands
    int depth;                  // slabs the register-staged path keeps in flight in registers
    launch_fn f16, f32, bf16;
    int fallback;               // -1, or (K split across the waves of a workgroup) the tile that takes
                                // operands this kernel does not serve: 2-byte aligned, ragged granules, ragged K
    int auto16, auto32;         // load paths (bit 0: direct loads, bit 1: register-staged, bit 2: register-staged on
                                // 2-byte aligned operands, bit 3: direct loads on 4-/8-byte aligned operands) for
                                // which the automatic selection considers this configuration, for 16-bit and for
                                // binary32 operands; 0: only when forced
    launch_fn stage16, stage_bf16;  // gemm_stage_kernel (null: none), see runs_stage
    launch_fn skew16, skew_bf16;    // the same for rows off the cache lines, see rows_off_lines
    double stage_slab, stage_a4;    // its slab time (microseconds per 64 k, one workgroup on a CU), on 4-/8-byte aligned operands over that
    int stage_from;                 // slabs from which it is ahead on whole ones
    int stage_most;                 // sixteenths of the CUs up to which it is ahead on whole slabs of 16-byte rows
    int skew_from;                  // slabs from which it straightens rows off the cache lines
};

#define GEMM_TILE_LAUNCHERS(BM, BN, WM, WN) \
    launch_tile<_Float16, BM, BN, WM, WN>, launch_tile<float, BM, BN, WM, WN>, launch_tile<__bf16, BM, BN, WM, WN>
#define GEMM_STAGE_LAUNCHERS(BM, BN, NST) \
    launch_stage<_Float16, BM, BN, NST>, launch_stage<__bf16, BM, BN, NST>, launch_skew<_Float16, BM, BN, NST + 1>, launch_skew<__bf16, BM, BN, NST + 1>
// The constants of this table and of estimate_cost are fitted, not derived: every configuration
// at 1..32 K slices was timed on MI355X with random operands (so at the ~1.5 GHz the part
// throttles to under sustained MFMA load) on the benchmark shapes and on 425 random shapes
// of all layouts and alignment classes (M, N in 128..9000, K in 64..50000), the model's terms were
// fitted to the times by least squares, and then adjusted to minimise the time lost by the
// model's pick against the best measured configuration (fit_cost_model.py; tune_sweep.py prints that ratio).  The
// slab times therefore absorb what the model has no term for (a lone workgroup's slab is bound
// by load latency, not by its MFMA work) and are not clock-peak figures.
// (64x128 before 128x64: the model often ties the two, and the tie goes to the first; 64x128 measures 4-8 % ahead)
const TileConfig kTiles[] = {
    {"t256x256", 256, 256, 1, 1.02, 1.02, 6.98, 6.98, 7.2, 0.83, 1.2, 1.05, 1.67, 1.25, 1,
     GEMM_TILE_LAUNCHERS(256, 256, 2, 2), -1, 15, 15, nullptr, nullptr, nullptr, nullptr, 0.0, 0.0, 0, 0, 0},
    {"t128x128", 128, 128, 2, 0.457, 0.868, 1.99, 3.64, 1.92, 1.39, 1.23, 0.817, 1.57, 1.3, 3,
     GEMM_TILE_LAUNCHERS(128, 128, 2, 2), -1, 15, 15, GEMM_STAGE_LAUNCHERS(128, 128, 4), 0.40, 1.435, 24, 15, 24},
    {"t64x64", 64, 64, 4, 0.265, 0.855, 0.495, 1.86, 1.27, 0.78, 1.07, 0.992, 1.65, 1.35, 4,
     GEMM_TILE_LAUNCHERS(64, 64, 2, 2), -1, 15, 15, GEMM_STAGE_LAUNCHERS(64, 64, 6), 0.20, 1.55, 16, 16, 32},
    {"t256x256w8", 256, 256, 1, 1.05, 1.05, 7.6, 7.6, 6.02, 0.812, 1.2, 0.915, 1.35, 1.15, 1,
     GEMM_TILE_LAUNCHERS(256, 256, 2, 4), -1, 15, 15, nullptr, nullptr, nullptr, nullptr, 0.0, 0.0, 0, 0, 0},
    {"t256x128", 256, 128, 1, 0.71, 0.71, 3.52, 3.52, 3.82, 0.637, 1.2, 1.09, 1.47, 1.3, 1,
     GEMM_TILE_LAUNCHERS(256, 128, 2, 2), -1, 15, 15, nullptr, nullptr, nullptr, nullptr, 0.0, 0.0, 0, 0, 0},
    {"t128x256", 128, 256, 1, 0.661, 0.661, 4.19, 4.19, 4.17, 1.78, 1.25, 0.864, 2.03, 1.3, 1,
     GEMM_TILE_LAUNCHERS(128, 256, 2, 2), -1, 15, 15, nullptr, nullptr, nullptr, nullptr, 0.0, 0.0, 0, 0, 0},
    {"t64x128", 64, 128, 2, 0.349, 0.512, 1.12, 1.86, 1.67, 1.11, 1.31, 0.884, 1.87, 1.3, 3,
     GEMM_TILE_LAUNCHERS(64, 128, 2, 2), -1, 15, 15, GEMM_STAGE_LAUNCHERS(64, 128, 5), 0.265, 1.585, 16, 16, 24},
    {"t128x64", 128, 64, 2, 0.371, 0.617, 1.14, 1.81, 1.33, 1.06, 1.31, 0.919, 1.84, 1.3, 3,
     GEMM_TILE_LAUNCHERS(128, 64, 2, 2), -1, 15, 15, GEMM_STAGE_LAUNCHERS(128, 64, 5), 0.285, 1.63, 16, 16, 24},
    // K split across the four waves of the workgroup (Section 5.3, small sizes); fitted on 16-byte aligned operands only
    {"k64x64", 64, 64, 4, 0.311, 0.854, 0.598, 2.02, 2.02, 0.781, 1.07, 0.992, 1.65, 1.0, 1,
     launch_ksplit<_Float16, 64, 64>, launch_ksplit<float, 64, 64>, launch_ksplit<__bf16, 64, 64>, 2, 1, 1, nullptr, nullptr, nullptr, nullptr, 0.0, 0.0, 0, 0, 0},
};
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);

// The kernel for small products (gemm_small_kernel.h) as a choice of its own beside the tiles.  To callers it is the
// smallest tile in one slice, on whose 64x64 pieces four of its blocks lie.
constexpr int kSmall = kNumTiles, kSmallAs = 2;
const TileConfig &tile_of(int choice) { return kTiles[choice == kSmall ? kSmallAs : choice]; }

std::mutex g_mutex;
int g_forced_tile = -1;    // -1: heuristic
int g_forced_splits = 0;   // 0: heuristic
bool g_forced_safe = false;
bool g_force_regload = false;  // ":regload" in a forced configuration: register-staged kernels whatever the alignment
int g_store_mode = 0;  // 0: by shape; 1: ":direct", C straight from registers; 2: ":staged", through LDS where possible
double g_cost_scale[GEMM_COST_TERMS] = {1.0, 1.0, 1.0, 1.0};
unsigned long long *g_trace = nullptr;  // profiling aid (gemm_set_phase_trace)
int64_t g_trace_records = 0;

// K-slice workspaces: one per (device, stream).  Work on one stream is ordered, so a stream's
// buffer is never used by two launches at once; different streams never share one.  A buffer
// that has become too small is retired, not freed (earlier launches may still use it and
// hipFree would wait for the whole device): gemm_shutdown() frees everything.  Sizes at least
// double on growth, so the retired buffers of a stream add up to less than its live one.
struct Workspace { void *ptr = nullptr; size_t bytes = 0; };
struct DeviceState {
    int num_cu = 0;
    void *static_scratch = nullptr;
    std::map<hipStream_t, Workspace> ws;
    std::vector<void *> retired;
};
std::map<int, DeviceState> g_dev;

// What the calling thread's last call ran.  Kept as it is and put into words by gemm_last_config: the text took longer
// (0.3 us) than the rest of the library's own part of a call.
struct LastCall {
    const char *type = nullptr, *special = nullptr, *tile = nullptr;  // special: "empty", "zero-fill", or null
    bool akc = false, bkc = false, small = false, safe = false, fixed_scratch = false;
    const char *path = nullptr;
    int splits = 0, tail = 0;  // tail: K-slices of the last tiles
    const char *kernel = nullptr;  // null: the special one
};
thread_local LastCall t_last;
thread_local char t_last_config[128];

int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Floats per row of a K-slice workspace: rows begin on 128-byte boundaries whatever N is, so the
// partial results go out, and are read back by the reduce pass, in 16-byte pieces.
int64_t ws_pitch(int64_t N) { return cdiv(N, 32) * 32; }
size_t ws_bytes(int64_t splits, int64_t M, int64_t N) { return (size_t)splits * (size_t)M * (size_t)ws_pitch(N) * sizeof(float); }

// Whether gemm_stage_kernel can straighten the rows of a K-contiguous operand: they begin on 16 bytes but off the cache lines.
// Where it does (skew_from): time without over with it, rows 16, 32 and 64 bytes off, 64 .. 256 workgroups, both operands
// K-contiguous or one: K = 512 0.88 .. 0.96 on all tiles (a longer start, one image more); K = 1024 64x64 0.89 .. 0.99, the others
// 0.97 .. 1.08; K = 2048 64x64 1.01 .. 1.07, the others 1.02 .. 1.19; K = 4096 64x64 1.05 .. 1.13, the others 1.05 .. 1.27.
bool rows_off_lines(const void *p, int64_t ld, int64_t rows) { return (uintptr_t)p % 128 == 0 && ld % 8 == 0 && ld % 64 != 0 && rows >= GPR; }

// Whether a launch on direct loads (16-bit operands, load path 0 or 3) runs gemm_stage_kernel: at most one workgroup per CU,
// and enough slabs to pay for its longer start, 0.5 us.  Time of gemm_tile_kernel over that of gemm_stage_kernel, geometric mean
// of the four layouts, launches back to back on operands that change from call to call:
//   whole slabs, 16-byte rows, K = 1536 and 4096: 64x64 1.37 and 1.59 with 256 workgroups, 64x128 1.15 and 1.23, 128x64 1.15 and
//   1.24; 128x128 1.07 and 1.13 with 160, 1.05 and 1.07 with 192, 1.03 and 1.05 with 240, and 0.98 .. 1.02 with 256 on one card,
//   0.90 (2048x2048x2048 20.9 -> 23.3 us) on another: a full chip of them is bound by power and by the loads of all CUs together,
//   not by what one workgroup waits for.  4- and 8-byte rows 1.0 .. 1.26 on every tile, with 256 workgroups too.
//   K = 512 0.88 .. 1.0, K = 768 0.9 .. 1.1 on all tiles.
//   ragged K, 72 .. 3080: 64x64 1.0 .. 1.4, the others 0.98 .. 1.1 with 96 .. 256 workgroups, but with both operands K-contiguous
//   1.01 at 72, 0.97 .. 0.99 from 136 to 1544 and 1.0 from 2056 on.
//   whole K, granules over the edge of an operand: K = 256 0.975 .. 1.0 (64x64 1.02), 512 1.0 (1.04), 768 1.02 .. 1.06 (1.12),
//   1024 and more 1.0 .. 1.5.
// Operands of more than 28 MiB are streamed rather than held by the caches.  A few workgroups do not keep enough loads in flight
// for that either way, and launches shorter than stage_from lose (128x3520x5120, eight slices of ten slabs, 128x128 15.8 -> 19.8);
// the others gain, over 420 products of 28 .. 300 MB with 100 .. 256 workgroups 1.49 on 64x64, 1.17 on 128x64, 1.14 on 64x128, 1.06 on
// 128x128, the last with a full chip too (8192x128x8192 40.6 -> 38.0, on another card 36.4 -> 34.3; 1024x1024x43264 141 -> 110).  One row
// of 128x128 tiles 1.10 at up to 15/16 of the CUs, over 249 products of up to 128 rows (all layouts, N and K from 1024 to 16384), but
// a full chip of them is behind, as it is on operands that the caches hold (stage_most), whatever the leading dimension: TN 128x8192x8192
// 35.6 -> 38.4 us, 128x8192x6144 29.3 -> 33.9, with rows of B 9216 elements apart 36.5 -> 38.5 and 29.7 -> 33.5; NT 128x4096x16384
// 42.9 -> 46.5.  A column of tiles is not: TN 8192x128x8192 40.4 -> 38.3, 8192x128x6144 35.6 -> 34.0.
// Below 2.5 MiB they stay in the L2s from call to call, and the ring's one slab ahead is enough: 256x512x1024 5.8 -> 6.3,
// 512x512x1024 5.9 -> 6.3, but 768x512x1024 8.4 -> 6.6.
// ragged: K or granules, as measured above (operands that gemm_ksplit_kernel cannot take).
// Rows off the cache lines that are straightened (off_lines, from skew_from slabs on) cost nothing more on a full chip, in the ring they do:
// a full chip of 128x128 tiles 1.03 .. 1.10 at K = 2048, 1.07 .. 1.16 at 4096 (2048x2048x2048 with rows padded by 16 bytes
// 26.1 -> 23.7; 128x8192x8192 NT 45.3 -> 35.7).
bool runs_stage(const TileConfig &t, int64_t M, int64_t workgroups, int64_t slabs, int64_t K, bool ragged, int path, int64_t operand_bytes, bool off_lines, int num_cu)
{
    if (t.stage16 == nullptr || workgroups > num_cu) return false;
    const bool pays = 16 * workgroups <= t.stage_most * num_cu || (off_lines && slabs >= t.skew_from);
    if (operand_bytes > (28LL << 20)) return slabs >= t.stage_from && 8 * workgroups >= 3 * num_cu && (M > t.BM || pays);
    if (K % 64 != 0) return true;
    if (ragged) return slabs >= 8;
    return slabs >= t.stage_from && operand_bytes >= (5LL << 19) && (path == 3 || pays);
}

size_t tail_bytes(const TileConfig &t, int64_t sliced, int splits) { return (size_t)sliced * (size_t)splits * (size_t)(t.BM * t.BN) * sizeof(float); }

// microseconds that cutting the `sliced` last tiles into s slices saves, by the model's slab time: a fifth of the time the
// round gets shorter is kept back for what a part-filled chip gains in clock
double tail_gain(const TileConfig &t, int64_t sliced, int64_t KT, int s, bool f32)
{
    const double saved = (double)(KT - cdiv(KT, s)) * (f32 ? t.f32_alone : t.f16_alone);
    return 0.8 * saved - (5.0 + (double)tail_bytes(t, sliced, s) * (1.0 + 1.0 / s) / 3.8e6);
}

// K-slices for the tiles of a last round that fills at most half of the chip (1: none).  One workgroup per CU: a round
// takes as long with 15 tiles as with 256, so the tiles past the last full round are cut into as many slices as there are
// CUs for them, and a second pass sums their partial tiles (tail_reduce_kernel).  Taken where the part of the round it saves
// is worth more than the partial tiles (written, read once more, the launch of the pass).
int tail_slices(const TileConfig &t, int64_t tiles, int64_t KT, bool f32, int num_cu, size_t max_ws_bytes)
{
    const int64_t sliced = tiles % num_cu;
    if (t.wg_per_cu != 1 || tiles < num_cu || sliced == 0 || 2 * sliced > num_cu) return 1;
    int64_t s = num_cu / sliced < 16 ? num_cu / sliced : 16;
    if (s > KT / 4) s = KT / 4;  // at least four slabs each
    if (s < 2) return 1;
    s = cdiv(KT, cdiv(KT, s));   // no empty slices
    const size_t bytes = tail_bytes(t, sliced, (int)s);
    if (max_ws_bytes > 0 && bytes > max_ws_bytes) return 1;
    return tail_gain(t, sliced, KT, (int)s, f32) > 0.0 ? (int)s : 1;
}

// What estimate_cost prices, and what is the same for every configuration.
struct Problem {
    int64_t M, N, K, KT;
    bool f32;
    int path, k_contig, num_cu;  // path: 0 = direct-load kernels, 1 = register-staged loads, 2 = register-staged loads of operands
                                 // that are only 2-byte aligned (each 16-byte load is then split up by the memory pipeline),
                                 // 3 = direct-load kernels on operands that are 4- or 8-byte aligned (row pieces straddle cache lines)
                                 // k_contig: how many of A and B have K as their contiguous dimension (0..2); the misaligned
                                 // classes depend on it (a K-contiguous row is what straddles lines or gets its loads split)
    size_t max_ws_bytes;         // see choose_uncached, ksplit_ok too
    bool ksplit_ok;
    double bytes;        // of A and B
    double foot_factor;  // on the slab time, of operands that the XCDs' L2s hold
    double streamed;     // doublings of bytes beyond those from which the stage kernel's slabs come later, or 0

    Problem(int64_t M, int64_t N, int64_t K, int64_t KT, bool f32, int path, int k_contig, int num_cu, size_t max_ws_bytes, bool ksplit_ok)
        : M(M), N(N), K(K), KT(KT), f32(f32), path(path), k_contig(k_contig), num_cu(num_cu), max_ws_bytes(max_ws_bytes), ksplit_ok(ksplit_ok)
    {
        // Operands small enough to stay in the XCDs' L2s between and within calls are served faster than ones that come
        // from the memory side: the slab time falls, log-linearly in the bytes of A and B, from 1 x at kFootHi bytes to
        // kFootFactor x at kFootLo bytes and below (fitted on the paper's power-of-two sizes, where it decides between
        // one slice and several for the sizes up to 1024).
        static const double kStreamed = 60e6;
        static const double kFootLo = 2.23e+05, kFootHi = 1.52e+07, kFootFactor = 0.29;
        bytes = ((double)M * K + (double)K * N) * (f32 ? 4.0 : 2.0);
        foot_factor = bytes <= kFootLo ? kFootFactor
                      : (bytes >= kFootHi ? 1.0 : exp(log(kFootFactor) * (log(kFootHi) - log(bytes)) / (log(kFootHi) - log(kFootLo))));
        streamed = bytes > kStreamed ? log2(bytes / kStreamed) : 0.0;
    }
};

// K cut into at most `wanted` slices of `per` slabs: `count` of them are not empty
struct Slicing {
    int wanted = 1;
    int64_t per = 0, count = 0;
    Slicing() {}
    Slicing(int64_t KT, int wanted) : wanted(wanted), per(cdiv(KT, wanted)), count(cdiv(KT, per)) {}
};

// the pass that sums S slices
double reduce_cost(const Problem &p, int64_t S)
{
    if (S <= 1) return 0.0;
    return (1.51 + 0.0868 * (double)S) * g_cost_scale[GEMM_COST_FIXED] +
           (double)p.M * p.N * 4.0 * (double)(S + 1) / (3.8e+06 * g_cost_scale[GEMM_COST_HBM]);
}

// What estimate_cost cannot fall below for this tile in any number of slices, without the pass that sums them
double least_cost(const TileConfig &t, const Problem &p, int64_t tiles)
{
    const double t_hbm = (p.bytes + (double)p.M * p.N * 4.0) / (4.79e+06 * t.hbm_eff * g_cost_scale[GEMM_COST_HBM]);
    const double t_l2 = (double)tiles * (double)p.KT * (t.BM + t.BN) * 128.0 / (2.18e+07 * g_cost_scale[GEMM_COST_L2]);
    return 0.999999 * (2.68 * g_cost_scale[GEMM_COST_FIXED] + (t_hbm > t_l2 ? t_hbm : t_l2));  // (less what rounding may make of it)
}

// Estimated run time in microseconds of (tile, splits) on this shape.  Three floors: the
// MFMA work as scheduled on 256 CUs (rounds of resident workgroups, slab time depending on
// how many workgroups share a CU), HBM traffic for the unique bytes (limited by how many
// bytes the resident workgroups keep in flight), and L2->CU traffic for all the bytes the
// workgroups pull; plus launch/fill/drain and, with K slices, the reduce pass.
double estimate_cost(const TileConfig &t, const Problem &p, int64_t tiles, const Slicing &slices)
{
    static const double kLayA4[3] = {0.867, 1.0, 0.986};  // 16-bit, path 3, by k_contig
    static const double kLayA2[3] = {1.14, 1.0, 1.19};   // 16-bit, path 2
    const double *const scale = g_cost_scale;
    const bool f32 = p.f32;
    const int path = p.path, k_contig = p.k_contig;
    const int64_t per = slices.per, S = slices.count, W = tiles * S;
    const double slots = (double)p.num_cu * t.wg_per_cu;
    const double rounds = (double)cdiv(W, (int64_t)p.num_cu * t.wg_per_cu);
    const int64_t share = cdiv(W, p.num_cu) < t.wg_per_cu ? cdiv(W, p.num_cu) : t.wg_per_cu;
    const double alone = f32 ? t.f32_alone : t.f16_alone, full = f32 ? t.f32_full : t.f16_full;
    double slab = alone + (t.wg_per_cu > 1 ? (full - alone) * (double)(share - 1) / (t.wg_per_cu - 1) : 0.0);
    // slabs' worth of extra time for a ragged K beside its last slab's own: a guarded loop on path 1 and 2; on direct loads, which
    // have none, a fitted term all the same (with zero in binary32 the picks of 39 calls were 2 .. 4 % slower, with zero or one
    // in 16 bits those of 367 and 375 calls 0.6 % slower and the same)
    double tail = f32 ? (path == 3 ? 3.23 : 1.27) : (path == 3 ? 2.8 : 2.32);
    if (path == 3) slab *= f32 ? t.f32_a4 : t.f16_a4 * kLayA4[k_contig];
    if (path == 1 || path == 2) slab *= f32 ? 1.05 : (path == 2 ? t.f16_a2 * kLayA2[k_contig] : t.general);
    slab *= p.foot_factor;
    // (its slab time hardly depends on where the operands come from; where it runs it is not behind the other kernel, whose
    // time for small operands is the lower one; a ragged last slab is one more.  16-byte rows are priced alike wherever they begin, on
    // the cache lines or off them, so a shape has one pick, which gemm_query_config can tell: with a price of their own for rows off the
    // lines the 240 of 3176 drawn products with such rows that had another pick took 1.015 times as long; where an operand is
    // K-contiguous, and straightened or not, 1.026, where neither is, 0.97)
    if (!f32 && (path == 0 || path == 3) && runs_stage(t, p.M, W, per, p.K, !p.ksplit_ok, path, (p.M + p.N) * p.K * 2, false, p.num_cu)) {
        double stage = t.stage_slab * (path == 3 ? t.stage_a4 * kLayA4[k_contig] : 1.0);
        stage *= 1.0 + (t.BM + t.BN < 256 ? 0.35 : 0.1) * p.streamed;
        if (stage < slab) slab = stage;
        tail = 0.0;
    }
    if (path == 1 || path == 2) {
        // the register-staged path keeps `depth` slabs in flight per workgroup: a slab cannot take
        // less than that share of a global-load round trip
        // (binary32 slabs are bound by their MFMA time: measured within 5 % of the direct path)
        const double floor = 1.2 / ((double)share * t.depth);
        if (slab < floor) slab = floor;
        if (!f32) tail = 4.58;
    }
    slab *= scale[GEMM_COST_SLAB];
    double t_mfma = rounds * ((double)per * slab + t.fixed);
    if (slices.wanted == 1) {
        const int ts = tail_slices(t, tiles, p.KT, f32, p.num_cu, p.max_ws_bytes);
        if (ts > 1) t_mfma -= tail_gain(t, tiles % p.num_cu, p.KT, ts, f32);
    }
    if (p.K % (f32 ? 32 : 64) != 0) t_mfma += tail * slab;
    const double unique = p.bytes + (double)p.M * p.N * 4.0;
    const double resident = (double)W < slots ? (double)W : slots;
    double hbm_rate = resident * 1.5 * (t.BM + t.BN) * 128.0 / 0.848;  // bytes/us the workgroups keep in flight
    if (hbm_rate > 4.79e+06) hbm_rate = 4.79e+06;
    hbm_rate *= t.hbm_eff;
    const double t_hbm = unique / (hbm_rate * scale[GEMM_COST_HBM]);
    const double t_l2 = (double)W * (double)per * (t.BM + t.BN) * 128.0 / (2.18e+07 * scale[GEMM_COST_L2]);
    return 2.68 * scale[GEMM_COST_FIXED] + (t_mfma > t_hbm ? (t_mfma > t_l2 ? t_mfma : t_l2) : (t_hbm > t_l2 ? t_hbm : t_l2)) + reduce_cost(p, S);
}

// Products gemm_small_kernel is the fastest for: blocks for one round of CUs, and a K that sixteen waves request in a
// round or two.  Measured against the tile kernels' pick (M N from 64 64 to 1024 256, microseconds per launch back to back):
// binary32 K = 136 6.3 -> 3.6, 256 6.9 -> 4.2, 512 7.5 .. 9.6 -> 5.7 .. 6.4, 768 6.8 .. 10.8 -> 7.3 .. 8.7;
// 16 bits K = 136 4.3 -> 3.5, 512 4.4 .. 6.2 -> 3.5 .. 4.1, 768 5.2 .. 7.2 -> 3.9 .. 5.0, 1024 with both operands K-contiguous
// 5.8 .. 5.9 -> 5.7 .. 5.8, 2048 6.4 .. 9.0 -> 6.8 .. 10.2;
// K-contiguous rows on 2-byte boundaries, whose loads are split up, K = 136 5.2 -> 3.6, 512 5.9 -> 8.2, where the bases are not on
// words; where they are (words), K = 257 5.3 .. 6.2 -> 2.7 .. 3.7, 511 6.3 .. 7.3 -> 3.5 .. 4.8, 767 7.1 .. 8.6 -> 4.5 .. 6.4, 1151
// 7.8 .. 11.1 -> 5.6 .. 8.1 (neither operand K-contiguous 8.2 .. 10.5 -> 4.5 .. 7.4), 1279 8.0 .. 10.6 -> 6.3 .. 9.3, the nearest 9.0 -> 8.7.
// Twice the blocks lose 10 % and more at any K.  Over 1202 calls inside the rule (all layouts, alignments and types, extents from
// 1, from 1x8192 to 8192x32) the time is 0.70 of the tile kernels' in the geometric mean; the slowest are K <= 32, where most of
// the waves have nothing to do (3.2 -> 3.4).
bool serves_small(int64_t M, int64_t N, int64_t K, bool f32, int path, int k_contig, bool words, int num_cu)
{
    if (cdiv(M, 32) * cdiv(N, 32) > num_cu) return false;
    return K <= (f32 ? 512 : path == 2 ? (words ? 1152 : (k_contig > 0 ? 256 : 768)) : 768);
}

// Whether it is bases on words that bring the small kernel in: a class of their own for recorded picks, because bases off the words
// leave the tile kernels to choose from, and a pick of either kind is none for the other.
bool by_words_only(int64_t M, int64_t N, int64_t K, bool f32, int path, int k_contig, bool words, int num_cu)
{
    return words && serves_small(M, N, K, f32, path, k_contig, true, num_cu) && !serves_small(M, N, K, f32, path, k_contig, false, num_cu);
}

// What can be forced, or traced, are the tile kernels: with any such setting the small kernel stays out, whether the
// rule above, a recorded pick or gemm_tune would run it (g_mutex held).
bool small_allowed()
{
    return g_forced_tile < 0 && g_forced_splits == 0 && !g_forced_safe && !g_force_regload && g_store_mode == 0 && g_trace == nullptr;
}

// K-slice counts the selection considers.  With powers of two alone the last doubling leaves up to half of the chip idle
// (600x912x16608, 40 tiles of 128x128: four slices 36.2 us, six 32.3).  A count between them is taken where it is predicted to be at
// least this much faster: the slices' runs then begin in the middle of an XCD's, and neighbours share less.  Over 500 products of
// up to 1.5e11 operations, the time with powers of two alone over that with all counts, for those whose pick changed: with no margin
// 1.065 (146, 22 of them 2.5 % and more slower), 3 % 1.070 (135, 19), 6 % 1.075 (118, 11), 10 % 1.091 (89, 7); over all products 1.015
// with any of them.  Binary32, whose slab times are steadier, 3 %.
const int kSlices[] = {1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16, 20, 24, 28, 32};
constexpr int kNumSlices = sizeof(kSlices) / sizeof(kSlices[0]);
bool power_of_two(int slices) { return (slices & (slices - 1)) == 0; }
double between_margin(int slices, bool f32) { return power_of_two(slices) ? 1.0 : (f32 ? 1.03 : 1.10); }

// max_ws_bytes: largest K-slice workspace the caller can provide (0 = no limit); automatic
// picks that would need more are not considered.
// ksplit_ok: the operands qualify for the kernels that split K across the waves of a workgroup
// words: rows begin in the middle of a word, and gemm_small_kernel can read them word by word
void choose_uncached(int64_t M, int64_t N, int64_t K, int64_t KT, bool f32, int path, int k_contig, int num_cu,
                     size_t max_ws_bytes, bool ksplit_ok, bool words, int &tile, int &splits)
{
    double best = 1e300;
    tile = g_forced_tile >= 0 ? g_forced_tile : 0;
    splits = 1;
    if (small_allowed() && serves_small(M, N, K, f32, path, k_contig, words, num_cu)) {
        tile = kSmall;
        return;
    }
    // a forced slice count beyond the number of slabs means one slab per slice
    const int forced = g_forced_splits > 0 ? (int)(g_forced_splits < KT ? g_forced_splits : KT) : 0;
    const Problem problem(M, N, K, KT, f32, path, k_contig, num_cu, max_ws_bytes, ksplit_ok);
    Slicing slicings[kNumSlices];
    int n = 0;
    for (const int s : kSlices) {
        const int cand = forced > 0 ? forced : s;
        if (cand > 1 && cand > KT) break;
        if (forced == 0 && cand > 1 && max_ws_bytes > 0 && ws_bytes(cand, M, N) > max_ws_bytes) break;
        slicings[n++] = Slicing(KT, cand);
        if (forced > 0) break;
    }
    for (int t = 0; t < kNumTiles; ++t) {
        if (g_forced_tile >= 0 && t != g_forced_tile) continue;
        if (g_forced_tile < 0 && kTiles[t].fallback >= 0 && !ksplit_ok) continue;
        if (g_forced_tile < 0 && !(((f32 ? kTiles[t].auto32 : kTiles[t].auto16) >> path) & 1)) continue;
        const int64_t tiles = cdiv(M, kTiles[t].BM) * cdiv(N, kTiles[t].BN);
        const double least = least_cost(kTiles[t], problem, tiles);
        for (int i = 0; i < n; ++i) {
            if (least + 0.999999 * reduce_cost(problem, slicings[i].count) >= best) break;  // (and more slices cost no less)
            const double c = estimate_cost(kTiles[t], problem, tiles, slicings[i]) * (forced > 0 ? 1.0 : between_margin(slicings[i].wanted, f32));
            if (c < best) { best = c; tile = t; splits = slicings[i].wanted; }
        }
    }
}

// The selection costs up to a hundred evaluations of the model (1 .. 2 us; of 16-bit products that fill the chip 0.4, for what cannot
// be the fastest any more is left out: 3.3 with every tile and count evaluated); calls repeat shapes, so the last picks
// are kept (g_mutex held; any change of the forced configuration or of the model's scales
// starts a new epoch and thereby empties the table).
struct Pick {
    int64_t M = -1, N = 0, K = 0;
    size_t max_ws = 0;
    uint64_t epoch = 0;
    int f32 = 0, path = 0, k_contig = 0, num_cu = 0, ksplit_ok = 0, words = 0, tile = 0, splits = 0;
};
Pick g_picks[64];
uint64_t g_epoch = 1;

// Picks found by measurement (gemm_tune): what a call is classified by -> (tile, K slices).  Consulted
// before the cost model unless a configuration or slice count is forced (g_mutex held).
struct ShapeKey {
    int64_t M, N, K;
    int f32, path, k_contig, num_cu, ksplit_ok;
    int words;  // by_words_only
    bool operator<(const ShapeKey &o) const
    {
        return std::tie(M, N, K, f32, path, k_contig, num_cu, ksplit_ok, words) <
               std::tie(o.M, o.N, o.K, o.f32, o.path, o.k_contig, o.num_cu, o.ksplit_ok, o.words);
    }
};
std::map<ShapeKey, std::pair<int, int>> g_tuned;

// What gemm_tune passes through a call: a configuration to run instead of the selection's (tile >= 0), and
// on return the call's classification (filled: the call reached the selection, i.e. it was not empty).
struct TuneRequest {
    int tile = -1, splits = 1;
    ShapeKey key{};
    bool filled = false;
    bool words = false;  // as for choose_uncached
};

void choose(int64_t M, int64_t N, int64_t K, int64_t KT, bool f32, int path, int k_contig, int num_cu,
            size_t max_ws_bytes, bool ksplit_ok, bool words, int &tile, int &splits)
{
    const uint64_t h = (uint64_t)M * 0x9E3779B97F4A7C15ull ^ (uint64_t)N * 0xC2B2AE3D27D4EB4Full ^
                       (uint64_t)K * 0x165667B19E3779F9ull ^ (uint64_t)(words * 64 + k_contig * 16 + path * 4 + f32 * 2 + ksplit_ok);
    if (g_forced_tile < 0 && g_forced_splits == 0 && !g_tuned.empty()) {
        const auto it = g_tuned.find(ShapeKey{M, N, K, (int)f32, path, k_contig, num_cu, (int)ksplit_ok,
                                              (int)by_words_only(M, N, K, f32, path, k_contig, words, num_cu)});
        if (it != g_tuned.end() && (it->second.first != kSmall || small_allowed()) && (max_ws_bytes == 0 || it->second.second == 1 ||
                                    ws_bytes(it->second.second, M, N) <= max_ws_bytes)) {
            tile = it->second.first;
            splits = it->second.second;
            return;
        }
    }
    Pick &e = g_picks[(h >> 32) & 63];
    if (e.M == M && e.N == N && e.K == K && e.max_ws == max_ws_bytes && e.epoch == g_epoch && e.f32 == (int)f32 &&
        e.path == path && e.k_contig == k_contig && e.num_cu == num_cu && e.ksplit_ok == (int)ksplit_ok && e.words == (int)words) {
        tile = e.tile;
        splits = e.splits;
        return;
    }
    choose_uncached(M, N, K, KT, f32, path, k_contig, num_cu, max_ws_bytes, ksplit_ok, words, tile, splits);
    e.M = M; e.N = N; e.K = K; e.max_ws = max_ws_bytes; e.epoch = g_epoch; e.f32 = f32; e.path = path; e.k_contig = k_contig;
    e.num_cu = num_cu; e.ksplit_ok = ksplit_ok; e.words = words; e.tile = tile; e.splits = splits;
}

bool bad_matrix(const void *p, int layout, int64_t &ld, int64_t rows, int64_t cols)
{
    if (layout != GEMM_ROW_MAJOR && layout != GEMM_COL_MAJOR) return true;
    const int64_t packed = layout == GEMM_ROW_MAJOR ? cols : rows;
    if (ld == 0) ld = packed;
    if (ld < packed) return true;
    if (rows > 0 && cols > 0 && p == nullptr) return true;
    return false;
}

// state of the current device (g_mutex held); asks the device for its CU count the first time
int device_state(DeviceState **out)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return GEMM_ERR_HIP;
    DeviceState &d = g_dev[dev];
    if (d.num_cu == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
            n = kDefaultNumCU;
        d.num_cu = n;
    }
    *out = &d;
    return GEMM_OK;
}

// workspace of (device, stream) as it is (g_mutex held)
Workspace &stream_workspace(DeviceState &d, hipStream_t stream)
{
    static thread_local char own_thread;  // hipStreamPerThread names another stream in every thread
    return d.ws[stream == hipStreamPerThread ? (hipStream_t)&own_thread : stream];
}

// The same, made at least `bytes` long
int get_workspace(DeviceState &d, hipStream_t stream, size_t bytes, void **out)
{
    Workspace &w = stream_workspace(d, stream);
    if (w.bytes < bytes) {
        const size_t want = bytes > 2 * w.bytes ? bytes : 2 * w.bytes;
        void *p = nullptr;
        if (hipMalloc(&p, want) != hipSuccess) {
            (void)hipGetLastError();
            if (want == bytes || hipMalloc(&p, bytes) != hipSuccess) {
                (void)hipGetLastError();
                return GEMM_ERR_WORKSPACE;
            }
            w.bytes = bytes;
        } else {
            w.bytes = want;
        }
        if (w.ptr) d.retired.push_back(w.ptr);
        w.ptr = p;
    }
    *out = w.ptr;
    return GEMM_OK;
}

// The same for the partial tiles of a last round, which a launch can do without: failing is no error, and a stream under
// capture has none, also where its workspace would do.  A graph that took it would share it with whatever its stream runs
// later, and with other graphs captured on that stream, whatever streams they are replayed on.  (Nor may a capture
// elsewhere in the process mind an allocation.)
bool get_tail_workspace(DeviceState &d, hipStream_t stream, size_t bytes, void **out)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusActive;
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    if (hipStreamIsCapturing(stream, &status) != hipSuccess || status != hipStreamCaptureStatusNone ||
        hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    const int rc = get_workspace(d, stream, bytes, out);
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    return rc == GEMM_OK;
}

// device address of this GPU's copy of `scratch` (g_mutex held); looked up once per device
int static_scratch(DeviceState &d, void **out)
{
    if (d.static_scratch == nullptr) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) {
            (void)hipGetLastError();
            return GEMM_ERR_HIP;
        }
        d.static_scratch = ptr;
    }
    *out = d.static_scratch;
    return GEMM_OK;
}

// T: operand type (bfloat16 runs the binary16 path with the other MFMA instruction, so it shares
// the binary16 slab times of the selection); TC: element type of C (float, or _Float16 for gemm_f16f16).
// noalloc: K-slice partials go to the fixed per-GPU array instead of a grown workspace.
template <typename T, typename TC>
int gemm_impl(int64_t M, int64_t N, int64_t K, const void *A, int layA, int64_t lda,
              const void *B, int layB, int64_t ldb, TC *C, int layC, int64_t ldc, void *stream_, bool noalloc = false,
              TuneRequest *tune = nullptr)
{
    constexpr bool f32 = sizeof(T) == 4;
    constexpr bool out16 = sizeof(TC) == 2;
    constexpr bool bf16 = std::is_same<T, __bf16>::value;
    const char *const type_name = f32 ? "f32" : (bf16 ? "bf16" : (out16 ? "f16f16" : "f16"));
    constexpr int64_t kMax = 2147483647LL - 256;
    if (M < 0 || N < 0 || K < 0) return GEMM_ERR_INVALID_ARG;
    if (lda < 0 || ldb < 0 || ldc < 0) return GEMM_ERR_INVALID_ARG;
    if (bad_matrix(A, layA, lda, M, K) || bad_matrix(B, layB, ldb, K, N) || bad_matrix(C, layC, ldc, M, N))
        return GEMM_ERR_INVALID_ARG;
    if (M > kMax || N > kMax || K > kMax) return GEMM_ERR_UNSUPPORTED;
    hipStream_t stream = (hipStream_t)stream_;
    if (M == 0 || N == 0) {
        t_last = LastCall();
        t_last.type = type_name;
        t_last.special = "empty";
        return GEMM_OK;
    }

    // A column-major C is the row-major N x M matrix C^T = B^T * A^T; a
    // transposed operand is the same buffer with the other layout flag.
    if (layC == GEMM_COL_MAJOR) {
        std::swap(A, B);
        std::swap(lda, ldb);
        const int la = layB ^ 1, lb = layA ^ 1;
        layA = la;
        layB = lb;
        std::swap(M, N);
        layC = GEMM_ROW_MAJOR;
    }

    if (K == 0) {
        const int64_t total = M * N;
        const int blocks = (int)(cdiv(total, 256) < 65536 ? cdiv(total, 256) : 65536);
        if (launch_kernel(fill_zero_kernel<TC>, dim3(blocks), dim3(256), stream, C, ldc, (int)M, (int)N) != hipSuccess)
            return GEMM_ERR_HIP;
        t_last = LastCall();
        t_last.type = type_name;
        t_last.special = "zero-fill";
        return GEMM_OK;
    }

    const bool akc = layA == GEMM_ROW_MAJOR;  // A(i,k) contiguous in k
    const bool bkc = layB == GEMM_COL_MAJOR;  // B(k,j) contiguous in k
    constexpr int EPC = Elem<T>::EPC, BK = Elem<T>::BK;
    // The direct global->LDS loads need 4-byte aligned addresses only (measured: bit-exact, and faster
    // than staging through registers); 16-byte aligned operands make every 128-byte row piece one cache
    // line and are the fastest class.  Operands that are only 2-byte aligned and leading dimensions too
    // long for 32-bit tile offsets take the register-staged kernels.
    const uintptr_t low_bits = (uintptr_t)A | (uintptr_t)B | (uintptr_t)(lda * (int64_t)sizeof(T)) |
                               (uintptr_t)(ldb * (int64_t)sizeof(T));
    bool aligned = (low_bits & 3) == 0;   // "aligned" from here on: served by the direct-load kernels
    // granules of an M/N-contiguous operand straddle its edge when the extent is not a multiple of the granule
    const bool ragged = (!akc && M % EPC != 0) || (!bkc && N % EPC != 0);
    // the direct loaders address a tile with 32-bit byte offsets from its origin
    const bool ld32 = 256 * lda * (int64_t)sizeof(T) < (1LL << 31) && 256 * ldb * (int64_t)sizeof(T) < (1LL << 31);
    if (!ld32) aligned = false;
    if (g_force_regload) aligned = false;
    // load path for the cost model: 0 direct loads on 16-byte aligned operands, 3 direct loads on 4- or
    // 8-byte aligned ones, 1 register-staged, 2 register-staged on 2-byte aligned operands
    const int path = aligned ? ((low_bits & 15) == 0 ? 0 : 3) : ((low_bits & 3) != 0 ? 2 : 1);

    // From here to the last launch under the lock: the selection reads the process-wide
    // overrides, and a K-sliced call's two launches must reach the stream back to back (another
    // host thread on the same stream would otherwise put its partials into the same workspace
    // between them).  Launches are asynchronous, so the lock is held for microseconds.
    std::lock_guard<std::mutex> lock(g_mutex);
    DeviceState *dev = nullptr;
    if (device_state(&dev) != GEMM_OK) return GEMM_ERR_HIP;
    const int num_cu = dev->num_cu;

    const int64_t KT = cdiv(K, BK);
    int tile, splits;
    const bool ksplit_ok = aligned && !ragged && K % BK == 0;
    // rows begin in the middle of a word, and gemm_small_kernel can read them word by word
    const bool words = !f32 && path == 2 && (((uintptr_t)A | (uintptr_t)B) & 3) == 0;
    if (tune) {
        tune->key = ShapeKey{M, N, K, (int)f32, path, (int)akc + (int)bkc, num_cu, (int)ksplit_ok,
                             (int)by_words_only(M, N, K, f32, path, (int)akc + (int)bkc, words, num_cu)};
        tune->filled = true;
        tune->words = words;
    }
    if (tune && tune->tile >= 0) {
        tile = tune->tile;
        splits = (int)(tune->splits < KT ? tune->splits : KT);
    } else {
        choose(M, N, K, KT, f32, path, (int)akc + (int)bkc, num_cu, noalloc ? (size_t)GEMM_NOALLOC_SCRATCH_BYTES : 0,
               ksplit_ok, words, tile, splits);
        // A stream under capture cannot be given a larger workspace: a pick in K-slices that needs one gives way to the best in
        // one slice, so that which calls can be captured does not depend on the model's constants.
        if (splits > 1 && !noalloc && tune == nullptr && g_forced_splits == 0 &&
            stream_workspace(*dev, stream).bytes < ws_bytes(cdiv(KT, cdiv(KT, splits)), M, N)) {
            hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
            if (hipStreamIsCapturing(stream, &status) != hipSuccess) (void)hipGetLastError();
            else if (status == hipStreamCaptureStatusActive)
                choose(M, N, K, KT, f32, path, (int)akc + (int)bkc, num_cu, 1, ksplit_ok, words, tile, splits);
        }
    }
    const bool small = tile == kSmall;
    if (tile_of(tile).fallback >= 0 && !ksplit_ok) tile = kTiles[tile].fallback;  // forced, but not served by that kernel
    const TileConfig &t = tile_of(tile);
    const int64_t tiles_m = cdiv(M, t.BM), tiles_n = cdiv(N, t.BN);
    int64_t kt_per_split = cdiv(KT, splits);
    splits = (int)cdiv(KT, kt_per_split);  // no empty slices
    if (tiles_m * tiles_n * splits > (1LL << 28)) return GEMM_ERR_UNSUPPORTED;

    KernelArgs a;
    a.A = A;
    a.B = B;
    a.lda = lda;
    a.ldb = ldb;
    a.M = (int)M;
    a.N = (int)N;
    a.K = (int)K;
    a.tiles_m = (int)tiles_m;
    a.tiles_n = (int)tiles_n;
    a.kt_per_split = (int)kt_per_split;
    a.splits = splits;
    a.whole_tiles = 0;
    a.tail_ws = nullptr;
    a.ld32 = ld32 ? 1 : 0;
    a.out16 = 0;
    a.stream_c = 0;
    a.safe = g_forced_safe ? 1 : 0;
    a.rows16_c = 0;
    a.stage_c = 0;
    a.trace = g_trace;
    a.trace_records = (int)(g_trace_records < (1LL << 30) ? g_trace_records : (1LL << 30));
    void *ws = nullptr;
    if (splits > 1) {
        const size_t need = ws_bytes(splits, M, N);
        int rc;
        if (noalloc) {
            // only a forced configuration can get here with more than the array holds
            if (need > (size_t)GEMM_NOALLOC_SCRATCH_BYTES) return GEMM_ERR_WORKSPACE;
            rc = static_scratch(*dev, &ws);
        } else {
            rc = get_workspace(*dev, stream, need, &ws);
        }
        if (rc != GEMM_OK) return rc;
        a.C = (float *)ws;
        a.ldc = ws_pitch(N);
        a.split_stride = M * ws_pitch(N);
        // slices and their rows begin on 128-byte boundaries (256-byte aligned base, padded rows)
        a.rows16_c = N < (1LL << 20) ? 1 : 0;
        a.stage_c = (a.rows16_c && g_store_mode != 1) ? 1 : 0;
    } else {
        a.C = (float *)C;
        a.ldc = ldc;
        a.split_stride = 0;
        a.out16 = out16 ? 1 : 0;
        // C through LDS in whole rows (16 bytes per lane): always for binary16 C (the direct stores
        // are 2 bytes per lane); for binary32 C when more than one round of tiles runs, where the
        // fewer store instructions pay (8192^3 -1 %); a single round is over sooner with the
        // stores leaving straight from the registers (2048^3 +4 %, 4096^3 binary32 +0.7 % staged)
        const bool can_stage = (uintptr_t)C % 16 == 0 && (ldc * (int64_t)sizeof(TC)) % 16 == 0 && ldc < (1LL << 20);
        const bool want_stage = out16 || tiles_m * tiles_n > (int64_t)num_cu * t.wg_per_cu;
        a.rows16_c = can_stage ? 1 : 0;
        a.stage_c = (can_stage && g_store_mode != 1 && (want_stage || g_store_mode == 2)) ? 1 : 0;
        // Non-temporal C stores (whole 128-byte lines only): measured 1-7 % faster when later rounds
        // of tiles are still reading A and B while C is written, or when C is small; 4-7 % slower
        // when one round of tiles writes more than the L2s hold in a single burst at the end.
        const bool lines = !out16 && ldc % 32 == 0 && (uintptr_t)C % 128 == 0;
        const bool rounds = tiles_m * tiles_n > (int64_t)num_cu * t.wg_per_cu;
        a.stream_c = (lines && (rounds || M * N * 4 <= (32LL << 20))) ? 1 : 0;
        // the tiles past the last full round of the chip cut into K-slices, unless one slice was asked for by name
        const int64_t tiles = tiles_m * tiles_n;
        const int tail = small || g_forced_splits != 0 ? 1 : tail_slices(t, tiles, KT, f32, num_cu, noalloc ? (size_t)GEMM_NOALLOC_SCRATCH_BYTES : 0);
        if (tail > 1 && (noalloc ? static_scratch(*dev, &ws) == GEMM_OK : get_tail_workspace(*dev, stream, tail_bytes(t, tiles % num_cu, tail), &ws))) {
            a.splits = tail;
            a.kt_per_split = (int)cdiv(KT, tail);
            a.whole_tiles = (int)(tiles - tiles % num_cu);
            a.tail_ws = (float *)ws;
        }
    }
    a.by_band = divisor(GM * tiles_n);
    a.by_last_rows = divisor(tiles_m % GM > 0 ? tiles_m % GM : 1);
    a.by_sliced = divisor(tiles_m * tiles_n - a.whole_tiles);
    hipError_t launch_rc;
    const char *kernel;
    if (small) {
        // binary32 in 16x16 blocks where those fit one round too and the sum is long enough to pay for four times the
        // workgroups (microseconds per launch, 32x32 -> 16x16 blocks: 256x256 NN K = 64 2.8 -> 3.6, 136 3.2 -> 3.3, 256 3.9 -> 3.5,
        // 512 5.9 -> 4.4; TN 256 4.4 -> 3.3; 512x512, two rounds and more, 4.1 -> 5.3)
        const bool blocks16 = f32 && K >= 192 && cdiv(M, 16) * cdiv(N, 16) <= num_cu;
        const int edge = blocks16 ? 16 : 32;
        a.tiles_m = (int)cdiv(M, edge);
        a.tiles_n = (int)cdiv(N, edge);
        const dim3 grid((unsigned)(a.tiles_m * a.tiles_n));
        kernel = blocks16 ? "gemm_small16_kernel" : "gemm_small_kernel";
        launch_rc = blocks16 ? launch_small16<float>(akc, bkc, grid, stream, a) : launch_small<T>(akc, bkc, grid, stream, a);
    } else {
        const dim3 grid((unsigned)work_grid((int)(tiles_m * tiles_n), a.whole_tiles, a.splits));
        launch_fn fn = f32 ? t.f32 : (bf16 ? t.bf16 : t.f16);
        const bool off_lines = (akc && rows_off_lines(A, lda, M)) || (bkc && rows_off_lines(B, ldb, N));
        const bool stage = !f32 && aligned && runs_stage(t, M, tiles_m * tiles_n * splits, kt_per_split, K, !ksplit_ok, path, (M + N) * K * (int64_t)sizeof(T), off_lines, num_cu);
        const bool skew = stage && off_lines && kt_per_split >= t.skew_from;
        if (skew) fn = bf16 ? t.skew_bf16 : t.skew16;
        else if (stage) fn = bf16 ? t.stage_bf16 : t.stage16;
        kernel = stage ? "gemm_stage_kernel" : (t.fallback >= 0 ? "gemm_ksplit_kernel" : "gemm_tile_kernel");
        launch_rc = fn(akc, bkc, aligned, grid, stream, a);
    }
    if (launch_rc != hipSuccess) {
        if (getenv("GEMM_VERBOSE"))
            fprintf(stderr, "gemm: launch of %s failed: %s\n", t.name, hipGetErrorString(launch_rc));
        return GEMM_ERR_HIP;
    }
    if (splits > 1) {
        const int64_t items = M * cdiv(N, 4);
        const int blocks = (int)(cdiv(items, 256) < 4096 ? cdiv(items, 256) : 4096);
        const int vec_c = ((uintptr_t)C % (4 * sizeof(TC)) == 0 && ldc % 4 == 0) ? 1 : 0;
        const hipError_t rc = launch_kernel(splitk_reduce_kernel<TC>, dim3(blocks), dim3(256), stream, (const float *)ws,
                                            (int64_t)(M * ws_pitch(N)), splits, (int)ws_pitch(N), C, ldc, (int)M, (int)N,
                                            vec_c);
        if (rc != hipSuccess) return GEMM_ERR_HIP;
    } else if (a.whole_tiles > 0) {
        const dim3 grid((unsigned)(t.BM * t.BN / 1024), (unsigned)(tiles_m * tiles_n - a.whole_tiles));
        const int vec_c = ((uintptr_t)C % (4 * sizeof(TC)) == 0 && ldc % 4 == 0) ? 1 : 0;
        const hipError_t rc = launch_kernel(tail_reduce_kernel<TC>, grid, dim3(256), stream, (const float *)ws, a.splits, a.whole_tiles,
                                            (int)tiles_m, (int)tiles_n, a.by_band, a.by_last_rows, t.BM, t.BN, C, ldc, (int)M, (int)N, vec_c);
        if (rc != hipSuccess) return GEMM_ERR_HIP;
    }
    t_last = LastCall{type_name, nullptr, t.name, akc, bkc, small, a.safe != 0, noalloc && a.splits > 1,
                      aligned ? (path == 0 ? "aligned" : "aligned4") : "general", splits, a.whole_tiles > 0 ? a.splits : 0, kernel};
    return GEMM_OK;
}

// Per-size tuning by measurement (Section 5.3 searches the configurations exhaustively per input size and
// keeps the best): runs the call once as it is, then times candidate (tile, K slices) pairs on the caller's
// operands, stream and device -- the cost model's `max_candidates` cheapest, or all -- and records the fastest
// for calls that classify alike.  Blocks the host on the stream; C ends up holding the product.
template <typename T, typename TC>
int tune_impl(int64_t M, int64_t N, int64_t K, const void *A, int layA, int64_t lda, const void *B, int layB, int64_t ldb,
              TC *C, int layC, int64_t ldc, void *stream_, int max_candidates, char *buf, int buflen)
{
    if (!buf || buflen <= 0 || max_candidates < 0) return GEMM_ERR_INVALID_ARG;
    constexpr int BK = Elem<T>::BK;
    hipStream_t stream = (hipStream_t)stream_;
    TuneRequest req;
    int rc = gemm_impl<T, TC>(M, N, K, A, layA, lda, B, layB, ldb, C, layC, ldc, stream_, false, &req);
    if (rc != GEMM_OK) return rc;
    if (!req.filled) {  // nothing to multiply
        snprintf(buf, (size_t)buflen, "none");
        return GEMM_OK;
    }
    const ShapeKey key = req.key;
    const int64_t KT = cdiv(key.K, BK);
    std::vector<std::tuple<double, int, int>> cand;
    {
        std::lock_guard<std::mutex> lock(g_mutex);
        if (small_allowed() && serves_small(key.M, key.N, key.K, key.f32 != 0, key.path, key.k_contig, req.words, key.num_cu)) cand.emplace_back(0.0, kSmall, 1);
        const Problem problem(key.M, key.N, key.K, KT, key.f32 != 0, key.path, key.k_contig, key.num_cu, 0, key.ksplit_ok != 0);
        for (int t = 0; t < kNumTiles; ++t) {
            if (kTiles[t].fallback >= 0 && !key.ksplit_ok) continue;
            const int64_t tiles = cdiv(key.M, kTiles[t].BM) * cdiv(key.N, kTiles[t].BN);
            for (const int s : kSlices) {
                if (s > 1 && s > KT) break;
                cand.emplace_back(estimate_cost(kTiles[t], problem, tiles, Slicing(KT, s)) * between_margin(s, problem.f32), t, s);
            }
        }
    }
    std::sort(cand.begin(), cand.end());
    if (max_candidates > 0 && (size_t)max_candidates < cand.size()) cand.resize((size_t)max_candidates);

    // One pass: `head` untimed launches of the first candidate, then every candidate of `list` gets `warm` untimed and
    // `timed` timed launches between two events of its own; everything is enqueued back to back and the host waits once
    // at the end, so the GPU never idles inside a pass (it lowers its clock within microseconds of idling, and whatever
    // is timed next -- the first candidate after a wait -- would be timed slow).
    // Returns (milliseconds per launch, tile, slices) of the candidates that ran.
    typedef std::vector<std::tuple<float, int, int>> timing_list;
    auto pass = [&](const timing_list &list, int head, int warm, int timed, timing_list &out) {
        std::vector<hipEvent_t> ev(2 * list.size(), nullptr);
        std::vector<char> ran(list.size(), 0);
        bool events_ok = true;
        for (auto &e : ev) events_ok = events_ok && hipEventCreate(&e) == hipSuccess;
        for (size_t c = 0; events_ok && c < list.size(); ++c) {
            req.tile = std::get<1>(list[c]);
            req.splits = std::get<2>(list[c]);
            const int untimed = warm + (c == 0 ? head : 0);
            bool ok = true;
            for (int i = 0; i < untimed + timed && ok; ++i) {
                if (i == untimed) ok = hipEventRecord(ev[2 * c], stream) == hipSuccess;
                ok = ok && gemm_impl<T, TC>(M, N, K, A, layA, lda, B, layB, ldb, C, layC, ldc, stream_, false, &req) == GEMM_OK;
            }
            ran[c] = ok && hipEventRecord(ev[2 * c + 1], stream) == hipSuccess;
        }
        if (events_ok) events_ok = hipStreamSynchronize(stream) == hipSuccess;
        for (size_t c = 0; events_ok && c < list.size(); ++c) {
            float ms = 0.0f;
            if (ran[c] && hipEventElapsedTime(&ms, ev[2 * c], ev[2 * c + 1]) == hipSuccess)
                out.emplace_back(ms / (float)timed, std::get<1>(list[c]), std::get<2>(list[c]));
        }
        for (auto &e : ev)
            if (e) (void)hipEventDestroy(e);
        (void)hipGetLastError();   // e.g. a candidate with no memory for its slices, or a stream under capture
    };
    // Without a limit every tile is timed in 1, 2, 4 .. 32 slices, and behind the model's favourite, which may have another count;
    // the counts between are timed around the four fastest only (all of them everywhere: 48 ms instead of 21 at 1536x1024x2048,
    // 3.3 s instead of 1.3 at 8192^3).
    timing_list all, first, finalists, second;
    for (const auto &c : cand)
        if (max_candidates > 0 || all.empty() || power_of_two(std::get<2>(c))) all.emplace_back(0.0f, std::get<1>(c), std::get<2>(c));
    // Six timed launches per candidate, behind 40 untimed ones of the model's favourite.  Then the four fastest and
    // the model's favourite again, twice in turn with 24 launches each, the better take of each kept: short kernels
    // time +-20 % on six launches, and a pick that is not measurably faster than the model's should not replace it.
    pass(all, 40, 2, 6, first);
    std::sort(first.begin(), first.end());
    if (first.size() > 4) first.resize(4);
    if (max_candidates == 0) {
        timing_list between;
        for (const auto &c : cand) {
            const int s = std::get<2>(c);
            bool near = false;
            for (const auto &f : first) near = near || (std::get<1>(f) == std::get<1>(c) && s < 2 * std::get<2>(f) && 2 * s > std::get<2>(f));
            if (near && !power_of_two(s) && !(std::get<1>(c) == std::get<1>(all[0]) && s == std::get<2>(all[0])))
                between.emplace_back(0.0f, std::get<1>(c), s);
        }
        if (!between.empty()) pass(between, 40, 2, 6, first);
        std::sort(first.begin(), first.end());
        if (first.size() > 4) first.resize(4);
    }
    finalists = first;
    bool has_model = false;
    for (const auto &f : first) has_model = has_model || (std::get<1>(f) == std::get<1>(all[0]) && std::get<2>(f) == std::get<2>(all[0]));
    if (!has_model && !first.empty()) finalists.push_back(all[0]);
    {
        timing_list twice = finalists;
        twice.insert(twice.end(), finalists.begin(), finalists.end());
        timing_list takes;
        pass(twice, 40, 3, 24, takes);
        for (const auto &f : finalists) {
            float best_ms = -1.0f;
            for (const auto &t : takes)
                if (std::get<1>(t) == std::get<1>(f) && std::get<2>(t) == std::get<2>(f) && (best_ms < 0.0f || std::get<0>(t) < best_ms))
                    best_ms = std::get<0>(t);
            if (best_ms >= 0.0f) second.emplace_back(best_ms, std::get<1>(f), std::get<2>(f));
        }
    }
    std::sort(second.begin(), second.end());
    int best_tile = -1, best_splits = 1;
    if (!second.empty()) {
        best_tile = std::get<1>(second[0]);
        best_splits = std::get<2>(second[0]);
    }
    if (best_tile < 0) return GEMM_ERR_HIP;
    {
        std::lock_guard<std::mutex> lock(g_mutex);
        const int64_t per = cdiv(KT, best_splits);
        g_tuned[key] = std::make_pair(best_tile, (int)cdiv(KT, per));
        ++g_epoch;
    }
    // the product, by the configuration just recorded (unless one is forced)
    rc = gemm_impl<T, TC>(M, N, K, A, layA, lda, B, layB, ldb, C, layC, ldc, stream_);
    const int64_t per = cdiv(KT, best_splits);
    snprintf(buf, (size_t)buflen, "%s:s%d", tile_of(best_tile).name, (int)cdiv(KT, per));
    return rc;
}

}  // namespace

extern "C" {

int gemm_f32(int64_t M, int64_t N, int64_t K, const float *A, int layoutA, int64_t lda,
             const float *B, int layoutB, int64_t ldb, float *C, int layoutC, int64_t ldc, void *hip_stream)
{
    return gemm_impl<float, float>(M, N, K, A, layoutA, lda, B, layoutB, ldb, C, layoutC, ldc, hip_stream);
}

int gemm_f16f32(int64_t M, int64_t N, int64_t K, const uint16_t *A, int layoutA, int64_t lda,
                const uint16_t *B, int layoutB, int64_t ldb, float *C, int layoutC, int64_t ldc,
                void *hip_stream)
{
    return gemm_impl<_Float16, float>(M, N, K, A, layoutA, lda, B, layoutB, ldb, C, layoutC, ldc, hip_stream);
}

int gemm_f16f16(int64_t M, int64_t N, int64_t K, const uint16_t *A, int layoutA, int64_t lda,
                const uint16_t *B, int layoutB, int64_t ldb, uint16_t *C, int layoutC, int64_t ldc,
                void *hip_stream)
{
    return gemm_impl<_Float16, _Float16>(M, N, K, A, layoutA, lda, B, layoutB, ldb, (_Float16 *)C, layoutC, ldc,
                                         hip_stream);
}

int gemm_bf16f32(int64_t M, int64_t N, int64_t K, const uint16_t *A, int layoutA, int64_t lda,
                 const uint16_t *B, int layoutB, int64_t ldb, float *C, int layoutC, int64_t ldc,
                 void *hip_stream)
{
    return gemm_impl<__bf16, float>(M, N, K, A, layoutA, lda, B, layoutB, ldb, C, layoutC, ldc, hip_stream);
}

int gemm_f16f32_noalloc(int64_t M, int64_t N, int64_t K, const uint16_t *A, int layoutA, int64_t lda,
                        const uint16_t *B, int layoutB, int64_t ldb, float *C, int layoutC, int64_t ldc,
                        void *hip_stream)
{
    return gemm_impl<_Float16, float>(M, N, K, A, layoutA, lda, B, layoutB, ldb, C, layoutC, ldc, hip_stream, true);
}

int gemm_tune(int kind, int64_t M, int64_t N, int64_t K, const void *A, int layoutA, int64_t lda, const void *B, int layoutB,
              int64_t ldb, void *C, int layoutC, int64_t ldc, void *hip_stream, int max_candidates, char *buf, int buflen)
{
    switch (kind) {
    case GEMM_KIND_F32:
        return tune_impl<float, float>(M, N, K, A, layoutA, lda, B, layoutB, ldb, (float *)C, layoutC, ldc, hip_stream,
                                       max_candidates, buf, buflen);
    case GEMM_KIND_F16F32:
        return tune_impl<_Float16, float>(M, N, K, A, layoutA, lda, B, layoutB, ldb, (float *)C, layoutC, ldc, hip_stream,
                                          max_candidates, buf, buflen);
    case GEMM_KIND_F16F16:
        return tune_impl<_Float16, _Float16>(M, N, K, A, layoutA, lda, B, layoutB, ldb, (_Float16 *)C, layoutC, ldc,
                                             hip_stream, max_candidates, buf, buflen);
    case GEMM_KIND_BF16F32:
        return tune_impl<__bf16, float>(M, N, K, A, layoutA, lda, B, layoutB, ldb, (float *)C, layoutC, ldc, hip_stream,
                                        max_candidates, buf, buflen);
    default:
        return GEMM_ERR_INVALID_ARG;
    }
}

int gemm_tune_clear(void)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    g_tuned.clear();
    ++g_epoch;
    return GEMM_OK;
}

// One recorded pick per line: "<bytes per operand element> M N K <alignment class> <K-contiguous operands> <CUs>
// <whole slabs and granules> <tile> <K slices>", "small" if the small kernel runs as that tile, and "words" for the class that
// by_words_only tells; lines starting with '#' are comments.
int gemm_tune_save(const char *path)
{
    if (path == nullptr) return GEMM_ERR_INVALID_ARG;
    FILE *f = fopen(path, "w");
    if (f == nullptr) return GEMM_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lock(g_mutex);
    fprintf(f, "# gemm_tune picks: elem_bytes M N K class k_contig cus whole tile slices\n");
    for (const auto &e : g_tuned) {
        const ShapeKey &k = e.first;
        fprintf(f, "%d %lld %lld %lld %d %d %d %d %s %d%s%s\n", k.f32 ? 4 : 2, (long long)k.M, (long long)k.N, (long long)k.K, k.path,
                k.k_contig, k.num_cu, k.ksplit_ok, tile_of(e.second.first).name, e.second.second, e.second.first == kSmall ? " small" : "", k.words ? " words" : "");
    }
    return fclose(f) == 0 ? GEMM_OK : GEMM_ERR_INVALID_ARG;
}

int gemm_tune_load(const char *path)
{
    if (path == nullptr) return GEMM_ERR_INVALID_ARG;
    FILE *f = fopen(path, "r");
    if (f == nullptr) return GEMM_ERR_INVALID_ARG;
    std::map<ShapeKey, std::pair<int, int>> read;
    char line[256];
    int rc = GEMM_OK;
    while (rc == GEMM_OK && fgets(line, sizeof line, f) != nullptr) {
        if (line[0] == '#' || line[0] == '\n' || line[0] == 0) continue;
        long long M, N, K;
        int esz, path_, kc, cus, whole, slices;
        int end = 0;
        char name[32];
        if (sscanf(line, "%d %lld %lld %lld %d %d %d %d %31s %d%n", &esz, &M, &N, &K, &path_, &kc, &cus, &whole, name, &slices, &end) != 10 ||
            (esz != 2 && esz != 4) || M <= 0 || N <= 0 || K <= 0 || path_ < 0 || path_ > 3 || kc < 0 || kc > 2 || cus <= 0 ||
            (whole != 0 && whole != 1) || slices < 1 || slices > 32) {   // gemm_tune records 1 .. 32 slices
            rc = GEMM_ERR_INVALID_ARG;
            break;
        }
        int tile = -1;
        for (int i = 0; i < kNumTiles; ++i)
            if (strcmp(name, kTiles[i].name) == 0) tile = i;
        // behind the slices: "small", which then has to serve the class, "words", both in this order, or nothing; then a comment
        bool small = false, by_words = false, known = true;
        const char *rest = line + end;
        char word[8];
        for (int used = 0; known && sscanf(rest, "%7s%n", word, &used) == 1 && word[0] != '#'; rest += used) {
            known = (strcmp(word, "small") == 0 && !small && !by_words) || (strcmp(word, "words") == 0 && !by_words);
            small = small || strcmp(word, "small") == 0;
            by_words = by_words || strcmp(word, "words") == 0;
        }
        if (by_words && !by_words_only(M, N, K, esz == 4, path_, kc, path_ == 2, cus)) known = false;
        if (small && !(tile == kSmallAs && slices == 1 && serves_small(M, N, K, esz == 4, path_, kc, by_words, cus))) known = false;
        if (!known) tile = -1;
        else if (small) tile = kSmall;
        // a tile this build does not have, or one that does not serve the class, makes the file invalid as a whole
        if (tile < 0 || (tile_of(tile).fallback >= 0 && !whole)) {
            rc = GEMM_ERR_INVALID_ARG;
            break;
        }
        read[ShapeKey{M, N, K, esz == 4, path_, kc, cus, whole, (int)by_words}] = std::make_pair(tile, slices);
    }
    fclose(f);
    if (rc != GEMM_OK) return rc;   // nothing of a bad file is taken over
    std::lock_guard<std::mutex> lock(g_mutex);
    for (const auto &e : read) g_tuned[e.first] = e.second;
    ++g_epoch;
    return GEMM_OK;
}

int gemm_query_config_layouts(int elem_bytes, int64_t M, int64_t N, int64_t K, int aligned, int layoutA, int layoutB,
                              char *buf, int buflen)
{
    if ((elem_bytes != 2 && elem_bytes != 4) || M <= 0 || N <= 0 || K <= 0 || !buf || buflen <= 0)
        return GEMM_ERR_INVALID_ARG;
    if ((layoutA != GEMM_ROW_MAJOR && layoutA != GEMM_COL_MAJOR) || (layoutB != GEMM_ROW_MAJOR && layoutB != GEMM_COL_MAJOR))
        return GEMM_ERR_INVALID_ARG;
    const bool f32 = elem_bytes == 4;
    const int64_t BK = f32 ? Elem<float>::BK : Elem<_Float16>::BK;
    const int64_t KT = cdiv(K, BK);
    // K is the contiguous dimension of a row-major A (M x K) and of a column-major B (K x N)
    const int k_contig = (layoutA == GEMM_ROW_MAJOR ? 1 : 0) + (layoutB == GEMM_COL_MAJOR ? 1 : 0);
    int tile, splits;
    {
        std::lock_guard<std::mutex> lock(g_mutex);
        // 16 or more (or 1): direct loads, aligned; 8 or 4: direct loads on misaligned rows; 0: register-staged
        // (operand extents that are not multiples of the granule); 2: register-staged, 2-byte aligned
        const int path = (aligned == 1 || aligned >= 16) ? 0 : (aligned == 2 ? 2 : (aligned >= 4 ? 3 : 1));
        choose(M, N, K, KT, f32, path, k_contig, kDefaultNumCU, 0, (path == 0 || path == 3) && K % BK == 0, false, tile, splits);
    }
    const int64_t per = cdiv(KT, splits);
    splits = (int)cdiv(KT, per);  // no empty slices, as in the launch path
    snprintf(buf, (size_t)buflen, "%s:s%d", tile_of(tile).name, splits);
    return GEMM_OK;
}

int gemm_query_config(int elem_bytes, int64_t M, int64_t N, int64_t K, int aligned, char *buf, int buflen)
{
    return gemm_query_config_layouts(elem_bytes, M, N, K, aligned, GEMM_ROW_MAJOR, GEMM_ROW_MAJOR, buf, buflen);
}

int gemm_force_config(const char *name)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    ++g_epoch;
    if (name == nullptr || strcmp(name, "auto") == 0 || name[0] == 0) {
        g_forced_tile = -1;
        g_forced_splits = 0;
        g_forced_safe = false;
        g_store_mode = 0;
        g_force_regload = false;
        return GEMM_OK;
    }
    // "<tile|auto>[:s<slices>][:safe][:direct|:staged][:regload]"
    std::string s(name);
    int splits = 0, store_mode = 0;
    bool safe = false, regload = false;
    size_t colon;
    while ((colon = s.rfind(':')) != std::string::npos) {
        const std::string tail = s.substr(colon + 1);
        if (tail == "safe") {
            safe = true;
        } else if (tail == "regload") {
            regload = true;
        } else if (tail == "direct" || tail == "staged") {
            if (store_mode != 0) return GEMM_ERR_UNSUPPORTED;
            store_mode = tail == "direct" ? 1 : 2;
        } else {
            if (tail.size() < 2 || tail[0] != 's' || splits != 0) return GEMM_ERR_UNSUPPORTED;
            char *end = nullptr;
            const long v = strtol(tail.c_str() + 1, &end, 10);
            if (*end != 0 || v < 1 || v > 1024) return GEMM_ERR_UNSUPPORTED;
            splits = (int)v;
        }
        s = s.substr(0, colon);
    }
    int tile = -1;
    if (s != "auto") {
        for (int i = 0; i < kNumTiles; ++i)
            if (s == kTiles[i].name) tile = i;
        if (tile < 0) return GEMM_ERR_UNSUPPORTED;
    }
    g_forced_tile = tile;
    g_forced_splits = splits;
    g_forced_safe = safe;
    g_store_mode = store_mode;
    g_force_regload = regload;
    return GEMM_OK;
}

int gemm_set_phase_trace(void *device_buffer, int64_t workgroups)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    if (device_buffer != nullptr && workgroups <= 0) return GEMM_ERR_INVALID_ARG;
    ++g_epoch;
    g_trace = (unsigned long long *)device_buffer;
    g_trace_records = device_buffer ? workgroups : 0;
    return GEMM_OK;
}

int gemm_cost_model_scale(int term, double factor)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    ++g_epoch;
    if (term < 0) {
        for (double &x : g_cost_scale) x = 1.0;
        return GEMM_OK;
    }
    if (term >= GEMM_COST_TERMS || !(factor > 0.0)) return GEMM_ERR_INVALID_ARG;
    g_cost_scale[term] = factor;
    return GEMM_OK;
}

int gemm_num_configs(void) { return kNumTiles; }

const char *gemm_config_name(int i) { return (i >= 0 && i < kNumTiles) ? kTiles[i].name : nullptr; }

const char *gemm_last_config(void)
{
    const LastCall &l = t_last;
    if (l.type == nullptr) return "none";
    char tail[16] = "";
    if (l.tail > 1) snprintf(tail, sizeof tail, " tail%d", l.tail);
    if (l.special != nullptr)
        snprintf(t_last_config, sizeof t_last_config, "%s %s", l.type, l.special);
    else
        snprintf(t_last_config, sizeof t_last_config, "%s %s %c%c %s s%d%s%s%s%s", l.type, l.tile, l.akc ? 'N' : 'T', l.bkc ? 'T' : 'N', l.path,
                 l.splits, l.small ? " small" : "", l.safe ? " safe" : "", tail, l.fixed_scratch ? " static-scratch" : "");
    return t_last_config;
}

const char *gemm_last_kernel(void)
{
    const LastCall &l = t_last;
    if (l.type == nullptr) return "none";
    return l.special != nullptr ? l.special : l.kernel;
}

const char *gemm_status_string(int status)
{
    switch (status) {
    case GEMM_OK: return "ok";
    case GEMM_ERR_INVALID_ARG: return "invalid argument";
    case GEMM_ERR_HIP: return "HIP runtime or launch failure";
    case GEMM_ERR_UNSUPPORTED: return "unsupported size or configuration";
    case GEMM_ERR_WORKSPACE: return "split-K workspace allocation failed";
    default: return "unknown status";
    }
}

int gemm_shutdown(void)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    int rc = GEMM_OK;
    int cur = 0;
    (void)hipGetDevice(&cur);
    for (auto &kv : g_dev) {
        DeviceState &d = kv.second;
        if (d.ws.empty() && d.retired.empty()) continue;
        if (hipSetDevice(kv.first) != hipSuccess) { rc = GEMM_ERR_HIP; continue; }
        // hipFree waits for the work that may still use the buffer
        for (auto &w : d.ws)
            if (w.second.ptr && hipFree(w.second.ptr) != hipSuccess) rc = GEMM_ERR_HIP;
        for (void *p : d.retired)
            if (hipFree(p) != hipSuccess) rc = GEMM_ERR_HIP;
        d.ws.clear();
        d.retired.clear();
    }
    (void)hipSetDevice(cur);
    return rc;
}

}  // extern "C"
