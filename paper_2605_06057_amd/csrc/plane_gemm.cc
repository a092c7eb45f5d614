// Host side of the plane GEMM (csrc/lcma_plane_gemm.hpp): choice of tile and of the schedule (Sec. 3.2, Split-Group
// Parallelism), launch.
#include "host_common.h"

#include <algorithm>
#include <cstring>

#define LCMA_PG_DECL(NAME) extern "C" int lcma_launch_pg_##NAME(const lcma::PlaneGemmParams *p, void *stream);
LCMA_PG_DECL(fp8_t256_bf16)
LCMA_PG_DECL(fp8_t128_bf16)
LCMA_PG_DECL(fp8_t256_f16)
LCMA_PG_DECL(fp8_t128_f16)
LCMA_PG_DECL(f16_t256_f16)
LCMA_PG_DECL(f16_t128_f16)
LCMA_PG_DECL(f16_t256_f32)
LCMA_PG_DECL(f16_t128_f32)
LCMA_PG_DECL(bf16_t256_bf16)
LCMA_PG_DECL(bf16_t128_bf16)
#define LCMA_PP_DECL(NAME) extern "C" int lcma_launch_##NAME(const lcma::PlaneGemmParams *p, void *stream);
LCMA_PP_DECL(pp_kn_bf16)
LCMA_PP_DECL(pp_kn_f16)
LCMA_PP_DECL(ppn_bf16)
LCMA_PP_DECL(ppn_f16)
LCMA_PP_DECL(ppn_bf16_kn)
LCMA_PP_DECL(ppn_f16_kn)

extern "C" int lcma_launch_few_rows_sum_f16(const lcma::FewRowsParams *p, int rows, void *stream);
extern "C" int lcma_launch_few_rows_sum_bf16(const lcma::FewRowsParams *p, int rows, void *stream);
#define LCMA_FR_DECL(NAME) extern "C" int lcma_launch_few_rows_##NAME(const lcma::FewRowsParams *p, int n, void *stream);
LCMA_FR_DECL(f16_16)
LCMA_FR_DECL(f16_32)
LCMA_FR_DECL(f16_64)
LCMA_FR_DECL(bf16_16)
LCMA_FR_DECL(bf16_32)
LCMA_FR_DECL(bf16_64)

#define LCMA_SP_DECL(NAME) extern "C" int lcma_launch_plain_##NAME(const lcma::FewRowsParams *p, int grid, void *stream);
#define LCMA_SP_DECL2(NAME) extern "C" int lcma_launch_plain_##NAME(const lcma::PlaneGemmParams *p, void *stream);
LCMA_SP_DECL(f32_t32x32x32_k4)
LCMA_SP_DECL(f32_t32x32x32_k4t)
#define LCMA_SP_TYPE(TYPE)                                                                          \
    LCMA_SP_DECL(TYPE##_t32x32x64_k4)                                                               \
    LCMA_SP_DECL(TYPE##_t32x32x64_k4t)                                                              \
    LCMA_SP_DECL(TYPE##_t64x64x64_k4)                                                               \
    LCMA_SP_DECL(TYPE##_t64x64x64_k4t)                                                              \
    LCMA_SP_PAIRS(TYPE)
#define LCMA_SP_PAIRS(TYPE)                                                                         \
    LCMA_SP_DECL2(TYPE##_t64x128x64_k2)                                                             \
    LCMA_SP_DECL2(TYPE##_t64x128x64_k2t)                                                            \
    LCMA_SP_DECL2(TYPE##_t128x128x64_k2)                                                            \
    LCMA_SP_DECL2(TYPE##_t128x128x64_k2t)
LCMA_SP_TYPE(bf16)
LCMA_SP_TYPE(f16)

namespace lcma {

namespace {
const int kCUs = 256;
typedef int (*Launch)(const PlaneGemmParams *, void *);
Launch launcher(int kind, int tile) {
    switch (kind * 2 + (tile == 256)) {
#define LCMA_PG_TILES(KIND, TYPE, OUT)                                       \
    case KIND * 2 + 1: return lcma_launch_pg_##TYPE##_t256_##OUT;            \
    case KIND * 2: return lcma_launch_pg_##TYPE##_t128_##OUT;
        LCMA_PG_TILES(PG_FP8_BF16, fp8, bf16)
        LCMA_PG_TILES(PG_FP8_F16, fp8, f16)
        LCMA_PG_TILES(PG_F16, f16, f16)
        LCMA_PG_TILES(PG_BF16, bf16, bf16)
        LCMA_PG_TILES(PG_F16_OUT, f16, f16)
        LCMA_PG_TILES(PG_F16_F32, f16, f32)
    }
    return nullptr;
}
int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
// work-groups that run at one time: one 256 x 256 tile (128 KB of LDS) or two 128 x 128 tiles (64 KB each) per CU
int slots_of(int tile) { return tile == 256 ? kCUs : 2 * kCUs; }
int64_t tile_cols(int tile) { return tile == 64 ? 128 : tile; }
} // namespace

int64_t plane_gemm_scratch_bytes(int tile) { return (int64_t)slots_of(tile) * 2 * tile * tile * 4; }

namespace {
// Tile and schedule together, by the time the slowest work-group takes.  Whole tile-products run in rounds of as many work-groups as fit;
// a step of 128 bytes of K takes a + b f + c f^4 us when a share f of them has one (with few of them the memory side answers sooner, with
// many the clock falls), and longer by `off_a` and `off_w` of itself for every 128 lines of K where rows of A or of W do not start on 128-byte lines
// (each piece of such a row lies in two; the longer the rows, the less of the other half is still there), a round `more` besides, the launch and the first loads
// `start`, 100 MB of operands `memory`, and beyond 80 MB `far` more, 100 MB of products `products`.
// Plain products: all forms of 5880 products, 1 to 16384 rows, N and K 256 to 16384, three sets of operands in turn (with one set the operands
// of small products come from the L2, and what waits longest looks best: 1 x 1096 x 11840 11.1 us instead of 8.2).  The prices are those with which
// the choice loses least, not the nearest to each time (7 to 13 % off): it takes 1.007 of the time of the fastest form at the sizes of linear layers, 1.009 over all, without the
// workspace 1.007 and 1.008; priced with one set and one penalty for either operand, ranges without any, 1.014 and 1.024 (658 x 8696 x 4736, rows of A off
// lines, 96 us on 256 x 256 instead of 72; 5506 x 3616 x 15744, both off, 1026 in ranges instead of 744).  Batches of Algorithm 1 (2050,
// planes of 128 to 8192 rows) where they run, between the passes over memory (by themselves, one after the other, the ping-pong kernel is 10 % slower against the
// others: the clock), again with three sets in turn; FP8 products (700) behind the quantisation of A.  The choice takes 1.004 of the time of the whole call with the fastest
// kernel in 16 bit, 1.002 and 1.001 in FP8; with the prices before, which had a step of 5 or 12 % at 5120 tile-products, 1.007 (fp32 products 1.015),
// 1.007 and 1.002 (9536 x 4592 x 1584 <3,3,3;23> fp16 360 us with the small tile twice to a CU, 329 with the large one).  256 x 256 with a work-group each, which has a step less
// where their number is odd, was not among them: 2841 x 2576 x 1264 <4,4,4;49> bf16, 5 steps, 94 us twice to a CU, 97 in turn, 88.
// Without the 64 x 128 tile plain products take 1.09, without both tiles of lcma_kpair.hpp 1.27; without the small tile's form with two work-groups to a CU
// (PlaneGemm: many tile-products of few steps, 384 x 384 x 960 in 49 planes 17.9 us, 26.6 on KPair) 1.01 to 1.08.
struct StepPrice {
    double a, b, c, more, start, off_a, off_w, memory, far, products;
    double step(double f) const { return a + b * f + c * f * f * f * f; }
};
enum { WHOLE_256, KPAIR_128, TWO_128, KPAIR_64, STATIC_256, NARROW }; // 256 x 256 ping-pong, 128 x 128, the same twice to a CU, 64 x 128, 256 x 256 a work-group each, 256 x 128 ping-pong
const StepPrice kPlain[] = {{0.807, 0.447, 0.0, 7.43, 0.0, 0.0, 0.113, 8.24, 0.0}, {0.339, 0.0559, 0.0735, 3.92, 1.4, 0.13, 0.0683, 0.167, 19.2}, {0.758, 0.212, 0.0, 2.14, 0.15, 0.0739, 0.089, 0.0, 0.0}, {0.241, 0.0685, 0.0, 2.64, 1.42, 0.19, 0.167, 0.362, 21.5}, {1.067, 0.171, 0.484, 4.70, 0.0, 0.11, 0.11, 0.0, 0.0}, {0.466, 0.265, 0.0, 6.22, 0.0, 0.432, 0.0, 0.0, 11.6}};
const StepPrice kBatch[] = {{0.99, 0.0, 0.416, 3.54, 8.0, 0.0, 0.0, 0.0, 0.0, 4.21}, {0.296, 0.0, 0.181, 1.47, 0.0, 0.0, 0.0, 14.3, 0.0, 14.8}, {0.651, 0.0, 0.311, 0.0, 0.0, 0.0, 0.0, 10.5, 0.0, 10.9}, {0.161, 0.0, 0.149, 1.53, 0.0, 0.0, 0.0, 12.3, 0.0, 6.3}, {1.29, 0.0, 0.318, 0.0, 0.0, 0.0, 0.0, 9.08, 0.0, 15.1}};
const StepPrice kBatchF32[] = {{1.02, 0.0, 0.34, 5.42, 8.0, 0.0, 0.0, 0.0, 0.0, 3.6}, {0.239, 0.0, 0.255, 3.17, 1.62, 0.0, 0.0, 14.2, 0.0, 0.0}, {0.575, 0.101, 0.339, 2.43, 0.293, 0.0, 0.0, 8.63, 0.0, 0.0}, {0.145, 0.0, 0.164, 1.84, 2.09, 0.0, 0.0, 11.1, 0.0, 2.38}, {1.18, 0.167, 0.354, 2.43, 0.0, 0.0, 0.0, 5.43, 0.0, 8.29}};
const StepPrice kBatchFp8[] = {{1.12, 0.0118, 0.28, 1.11, 4.08, 0.0, 0.0, 6.91, 0.0, 12.7}, {0.353, 0.00691, 0.238, 0.563, 0.000211, 0.0, 0.0, 9.92, 0.0, 30.1}, {0.744, 0.0, 0.332, 0.0, 0.0, 0.0, 0.0, 12.5, 0.0, 13.2}, {0.211, 0.0, 0.231, 1.29, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0}, {1.32, 0.179, 0.24, 0.0, 0.0, 0.0, 0.0, 11.4, 0.0, 15.0}};
const StepPrice kFp8[] = {{1.07, 0.0, 0.309, 5.5, 0.0, 0.0, 0.0, 0.0, 0.0, 5.42}, {0.3, 0.162, 0.0286, 2.08, 0.0, 0.0, 0.0, 0.0, 0.0, 17.3}, {0.667, 0.45, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 8.92}, {0.241, 0.102, 0.000282, 0.99, 0.0, 0.0, 0.0, 0.0, 0.0, 30.0}, {1.32, 0.217, 0.238, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 17.3}};
struct Operands {
    bool off_a, off_w; // rows that do not start on 128-byte lines
    double mbytes, lines, products; // lines: of 128 bytes along K; products: MB of them
    double far() const { return std::max(0.0, mbytes - 80.0); } // (three sets of them in turn no longer fit the last-level cache)
};
Operands plain_operands(int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldw) { return Operands{lda % 64 != 0, ldw % 64 != 0, (double)(M + N) * (double)K * 2e-6, (double)K / 64.0, 0.0}; }
Operands planes_operands(int kind, int planes, int64_t rows, int64_t cols, int ny) {
    return Operands{false, false, (double)planes * (double)(rows + cols) * ny * 128e-6, (double)ny, (double)planes * (double)rows * (double)cols * (kind == PG_F16_F32 ? 4e-6 : 2e-6)};
}
double off_lines(const Operands &o, double off_a, double off_w) { return 1.0 + (o.off_a ? off_a : 0.0) + (o.off_w ? off_w : 0.0); }
double rounds_us(const StepPrice &q, int64_t jobs, int64_t slots, int64_t steps, const Operands &o) {
    const double line = 1.0 + (off_lines(o, q.off_a, q.off_w) - 1.0) * o.lines / 128.0, f = (double)(jobs % slots) / (double)slots;
    return q.start + 0.01 * (q.memory * o.mbytes + q.far * o.far() + q.products * o.products) + (double)(jobs / slots) * ((double)steps * line * q.step(1.0) + q.more) + (f > 0.0 ? (double)steps * line * q.step(f) + q.more : 0.0);
}
// What else there is (measured as above):
//   slices of K for work-groups of their own (128 x 128, plain 16-bit products of few tiles): the fp32 products of the slices are written and
//     added by a second kernel, 1.4 us, 0.64 a slice and 0.2 per MB (743 x 1400 x 7168, 66 tiles in three slices: 24.8 us, 43.8
//     in one piece; 1024 x 1024 x 14336 36.7 / 85; 512 x 4096 x 14336 61.8 / 87.7);
//   Split-Group ranges: 1.75 (FP8 2.0) a step on 256 x 256, 6 a tile-product and 65 for the pieces (882 x 5224 x 10368 126 us, 179 on 256 x 128).  On
//     128 x 128 neighbouring tiles start at different k and share little in L2, 0.95 a step, unless the ranges divide a tile evenly, 0.68; 2.9 and 1.5 a piece
//     of a tile (512 x 4096 x 14336 65.6 us, 255 x 8504 x 7296 71 against 44 without, 559 x 7184 x 9856 196 / 106).  Half of the workspace serves
//     them alone.  Batches at the older prices: in 16 bit they have ranges only where a workspace is larger than asked for; of 420 FP8 calls none took them.
// tile, schedule: 0 = choose.  low: tiles of 64 x 128 are offered.  Returns microseconds (0 when nothing fits).
enum { STATIC = 1, RANGES = 2, PERSIST = 3, SLICES = 4, TWO_PER_CU = 5 };
int64_t slice_steps(int64_t jobs, int ny) { return ceil_div(ny, std::max<int64_t>(1, std::min<int64_t>(kCUs / jobs, ny / 4))); }
double choose(int kind, int planes, int64_t rows, int64_t cols, int ny, int tile, int schedule, const Operands &o, bool low, int64_t scratch_bytes, int *best_tile,
              int *best_sched) {
    const bool fp8 = kind == PG_FP8_BF16 || kind == PG_FP8_F16;
    const StepPrice *const price = fp8 ? (planes > 1 ? kBatchFp8 : kFp8) : kind == PG_F16_F32 ? kBatchF32 : planes > 1 ? kBatch : kPlain;
    double best = 0.0;
    *best_tile = *best_sched = 0;
    for (int t : {256, 128, 64}) { // (64: 64 x 128)
        if (tile ? t != tile : t == 64 && !low) continue;
        const int64_t jobs = (int64_t)planes * ceil_div(rows, t) * ceil_div(cols, tile_cols(t));
        const int64_t even = ny > 2 ? (ny + 1) & ~1 : ny; // (kernels of two groups of waves round an odd number of steps up)
        for (int sc : {STATIC, RANGES, PERSIST, SLICES, TWO_PER_CU}) {
            if (schedule && sc != schedule && !(sc == TWO_PER_CU && schedule == STATIC)) continue;
            const bool pingpong = t == 256 && sc == PERSIST;
            if (t == 64 && sc != STATIC) continue;
            if (!schedule && (t == 128 ? sc == PERSIST : price == kPlain && t == 256 && sc == STATIC)) continue; // (128: the same kernel as STATIC; plain 256 x 256: never ahead by more than 1 %)
            if (sc == RANGES && scratch_bytes < plane_gemm_scratch_bytes(t)) continue;
            double cost;
            if (sc == RANGES) {
                const int64_t cap = ceil_div(jobs * ny, slots_of(t));
                const bool even_ranges = ny % (2 * cap) == 0;
                if (price == kPlain)
                    cost = t == 256 ? (double)cap * 1.75 * off_lines(o, 0.05, 0.175) + 6.0 * (double)jobs / kCUs + 65.0
                                    : (double)(2 * cap) * (even_ranges ? 0.682 : 0.946) * off_lines(o, 0.0, 0.123) + 2.9 + 1.46 * (double)kCUs / (double)jobs + 2.44 * 0.01 * o.far();
                else
                    cost = t == 256 ? (double)cap * (fp8 ? 2.0 : 1.75) + 6.0 * (double)jobs / kCUs + 65.0
                                    : (double)(2 * cap) * (even_ranges ? price[KPAIR_128].step(1.0) : 0.85) + 12.0 + 2.3 * (double)kCUs / (double)jobs;
            } else if (sc == SLICES) {
                if (t != 128 || planes > 1 || fp8 || kind == PG_F16_F32 || 2 * jobs > kCUs || ny < 8 || scratch_bytes < plane_gemm_scratch_bytes(256)) continue;
                const int64_t cap = slice_steps(jobs, ny), slices = ceil_div(ny, cap);
                StepPrice q = price[KPAIR_128];
                q.far = 4.62; // (more CUs at it)
                cost = rounds_us(q, jobs * slices, kCUs, (cap + 1) & ~(int64_t)1, o) + 1.35 + 0.641 * (double)slices + 0.2 * 65536e-6 * (double)(jobs * slices);
            } else if (sc == TWO_PER_CU) {
                // (one or two steps and one round of tiles stay on KPair, where they are one chain: 6.0 us, 4.7 here, both below a call's 6 on the host)
                if (t != 128 || (price == kPlain && ny <= 2 && jobs <= kCUs)) continue;
                cost = rounds_us(price[TWO_128], jobs, 2 * kCUs, ny, o);
            } else if (t < 256) {
                cost = rounds_us(price[t == 128 ? KPAIR_128 : KPAIR_64], jobs, kCUs, even, o);
            } else if (pingpong) {
                cost = rounds_us(price[WHOLE_256], jobs, kCUs, (ny + 1) & ~1, o);
            } else {
                cost = rounds_us(price[STATIC_256], jobs, kCUs, ny, o);
            }
            if (!*best_tile || cost < best) {
                best = cost;
                *best_tile = t;
                *best_sched = sc;
            }
        }
    }
    return best;
}
} // namespace

// Seconds of the batched stage of Algorithm 1 in 16 bit as plane_gemm runs it by now (fp32_out: products kept in fp32), for
// lcma_select_dataflow.
double batched_plane_gemm_seconds(bool fp32_out, int planes, int64_t rows, int64_t cols, int ny) {
    const int kind = fp32_out ? PG_F16_F32 : PG_F16;
    int t = 0, sc = 0;
    const double us = choose(kind, planes, rows, cols, ny, 0, tuning_schedule(), planes_operands(kind, planes, rows, cols, ny), true, 0, &t, &sc);
    return t ? 1e-6 * us : -1.0;
}

// The same as lcma_predict_unfused_seconds was published with, and as lcma_gemm_ws, whose contract names that function, compares it:
// steps of the slowest work-group at 1.62 us, 3.5 or 5 more for every tile it works through, a pair of small tiles at 0.76 of a
// large one, 80 for the pieces of the Split-Group ranges, whole tiles only.  The kernels are up to a fifth faster by now.
double plane_gemm_seconds(int planes, int64_t rows, int64_t cols, int ny, int64_t scratch_bytes) {
    const int schedule = tuning_schedule();
    double best = -1.0;
    for (int t : {256, 128}) {
        if (planes > 1 && (rows % t || cols % t)) continue;
        const int64_t jobs = (int64_t)planes * ceil_div(rows, t) * ceil_div(cols, t);
        for (int sc : {1, 2, 3}) {
            if (schedule && sc != schedule) continue;
            if (sc == 2 && scratch_bytes < plane_gemm_scratch_bytes(t)) continue;
            const double rounds = (double)ceil_div(jobs, slots_of(t));
            const double steps = sc == 2 ? (double)ceil_div(jobs * ny, slots_of(t)) + 80.0 : rounds * (ny + (sc == 3 && rounds > 1 ? 3.5 : 5.0));
            const double cost = steps * (t == 256 ? 1.0 : 0.76) * (sc == 2 ? 1.05 : 1.0);
            if (best < 0.0 || cost < best) best = cost;
        }
    }
    return best < 0.0 ? -1.0 : best * 1.62e-6;
}

// Column panels of the tile order: `wide` tiles, or the widest of one, two or three less that leaves no narrower panel at the
// end (28 columns of tiles as 4 x 7 instead of 3 x 8 + 4: the batched stage at the FFN shape 1 % faster).
static int panel_of(int nz, int wide) {
    int panel = tuning_panel() == 8 ? wide : tuning_panel();
    if (panel == wide && nz % wide)
        for (int w : {wide - 1, wide - 2, wide - 3})
            if (nz % w == 0) {
                panel = w;
                break;
            }
    return panel < nz ? panel : nz;
}

// p: operands, extents, pitches, plane strides, ny, n_row_b filled in by the caller for `planes` planes of rows x cols
// (padded sizes; a tile may hang over the end of a plane).  tile: 256 or 128, 0 = choose.
// schedule: 0 = choose, 1 = one tile-product per work-group, 2 = Split-Group ranges (needs `scratch` of
// plane_gemm_scratch_bytes(tile) bytes), 4 = slices of K (plain 16-bit products), 3 = persistent work-groups that each take every units-th whole tile-product.
lcma_status plane_gemm(const char *who, int kind, PlaneGemmParams p, int planes, int64_t rows, int64_t cols, int tile,
                       int schedule, void *scratch, int64_t scratch_bytes, void *stream) {
    const int forced = tuning_schedule();
    if (forced) schedule = forced;
    int best_tile = 0, best_sched = 0;
    choose(kind, planes, rows, cols, p.ny, tile, schedule, kind == PG_BF16 || kind == PG_F16_OUT ? plain_operands(rows, cols, (int64_t)p.ny * 64, p.lda_b / 2, p.ldb_b / 2) : planes_operands(kind, planes, rows, cols, p.ny), true, scratch ? scratch_bytes : 0, &best_tile, &best_sched);
    if (!best_tile) {
        if (schedule == 2)
            return fail(LCMA_ERR_ARG, "%s: the Split-Group schedule needs %lld bytes of scratch", who,
                        (long long)plane_gemm_scratch_bytes(tile ? tile : 256));
        return fail(LCMA_ERR_SHAPE, "%s: no tile and schedule fit", who);
    }
    tile = best_tile;
    schedule = best_sched;
    Launch launch = launcher(kind, tile);
    if (!launch) return fail(LCMA_ERR_NOKERNEL, "%s: no plane GEMM kernel of kind %d", who, kind);
    if (!p.tail_b) p.tail_b = 128; // whole steps
    p.nx = (int32_t)ceil_div(rows, tile);
    p.nz = (int32_t)ceil_div(cols, tile_cols(tile));
    const int64_t jobs = (int64_t)planes * p.nx * p.nz, total = jobs * p.ny;
    if (total >= ((int64_t)1 << 31)) return fail(LCMA_ERR_SHAPE, "%s: too many tile steps", who);
    p.jobs = (int32_t)jobs;
    p.panel = panel_of(p.nz, 8);
    const int slots = slots_of(tile);
    p.interleave = 0;
    if (schedule == SLICES) {
        p.cap = slice_steps(jobs, p.ny);
        p.units = (int32_t)(2 * jobs * ceil_div(p.ny, p.cap)); // (groups of four waves, two to a work-group)
        p.interleave = 3;
        p.partial = scratch;
    } else if (schedule == PERSIST) { // persistent work-groups, whole tile-products u, u + units, ...
        p.units = (int32_t)(jobs < slots ? jobs : slots);
        p.cap = p.ny;
        // batches of planes: rounds of consecutive tile-products; one product: an eighth of them per XCD (see
        // PlaneGemm::run), which needs the same number of work-groups on every XCD
        p.interleave = planes > 1 || (p.units & 7) ? 1 : 2;
        p.partial = nullptr;
    } else if (schedule == RANGES) {
        p.units = (int32_t)(total < slots ? total : slots);
        p.cap = ceil_div(total, p.units);
        p.units = (int32_t)ceil_div(total, p.cap); // no idle work-group at the end
        p.partial = scratch;
    } else {
        p.units = (int32_t)jobs;
        p.cap = p.ny;
        p.partial = nullptr;
        p.interleave = schedule == TWO_PER_CU ? 4 : tile == 64 ? 5 : 0;
    }
    int err = launch(&p, stream);
    if (!err && schedule == SLICES) { // the fp32 products of the slices lie one after the other, in whole tiles
        FewRowsParams q;
        std::memset(&q, 0, sizeof q);
        q.C = p.C;
        q.ldc_b = p.ldc_b;
        q.n_row_b = p.n_row_b;
        q.row_blocks = p.nx;
        q.block_rows = tile;
        q.slices = p.units / (2 * p.jobs);
        q.partial_ld = p.nz * tile;
        q.partial = p.partial;
        err = (kind == PG_BF16 ? lcma_launch_few_rows_sum_bf16 : lcma_launch_few_rows_sum_f16)(&q, (int)rows, stream);
    }
    if (err) return fail(LCMA_ERR_HIP, "%s: plane GEMM launch failed with HIP error %d", who, err);
    return LCMA_OK;
}

// Microseconds of the plain product on the ping-pong kernel with tiles of 256 x tn (f: share of the CUs that a round fills), as
// the choice between it and the generated kernels was measured.  256 x 128: 0.52 + 0.38 f a
// step (K x N: 0.60 + 0.32 f, its fragments wait for their own reads) and 4 a round (K x N: 2048 x 4096 x 4096 62 against 87 for
// the generated kernel, 1024 x 4096 x 4096 50 / 56, 2048 x 4096 x 14336 210 / 284, 704 x 704 x 8000 80 / 98); 256 x 256: 0.80 + 0.72 f
// and 6 (K x N: 6144^3 394 / 495, 8192 x 14336 x 4096 704 / 863); 15 % more when rows do not start on
// 128-byte lines (5000 x 3000 x 1000 43 / 42), 30 % with N x K weights on the 256 x 128 tile (1178 x 2592 x 9952 130 / 104).
double plain_product_us(bool b_kn, int tn, int64_t M, int64_t N, int64_t K, bool off_line) {
    const int64_t ny = ceil_div(K, 64), jobs = ceil_div(M, 256) * ceil_div(N, tn), full = jobs / kCUs, rest = jobs % kCUs;
    const double line = !off_line ? 1.0 : tn == 128 && !b_kn ? 1.3 : 1.15;
    auto round = [&](double f) {
        return tn == 256 ? (double)((ny + 1) & ~(int64_t)1) * line * (0.80 + 0.72 * f) + 6.0
                         : (double)ny * line * (b_kn ? 0.60 + 0.32 * f : 0.52 + 0.38 * f) + 4.0;
    };
    return (double)full * round(1.0) + (rest ? round((double)rest / kCUs) : 0.0) + (tn == 256 ? 1.5 : 0.0);
}

// The plain 16-bit product C = A B (b_kn: B is K x N) or A W^T on the ping-pong kernels, for lcma_gemm, lcma_gemm_nt and lcma_gemm_ex
// (the same bits as the generated kernels: every element of C is one chain of 32x32x16 instructions over ascending k).
// Arguments are checked by the caller; K a multiple of 8.  Returns false, with nothing launched, when the generated kernel is
// predicted to take less than the `limit_us` given (tn, 256 or 128: this tile, whatever is predicted), or when padded offsets do not fit; else *err is the launch's HIP error.
bool plain_product(bool b_kn, int64_t M, int64_t N, int64_t K, const void *A, int64_t lda, const void *B, int64_t ldb, void *C, int64_t ldc,
                   int dtype, double limit_us, void *stream, int *err, int tn) {
    const int ny = (int)ceil_div(K, 64);
    auto cost = [&](int tn) { return plain_product_us(b_kn, tn, M, N, K, lda % 64 || ldb % 64); };
    if (!tn) {
        tn = cost(256) < cost(128) ? 256 : 128;
        if (cost(tn) >= limit_us) return false;
    }
    const int64_t lim = (int64_t)1 << 31, Mp = ceil_div(M, 256) * 256, Np = ceil_div(N, 256) * 256, Kp = (int64_t)(ny + 1) * 64;
    if (((Mp - 1) * lda + Kp) * 2 >= lim || (b_kn ? (Kp - 1) * ldb + Np : (Np - 1) * ldb + Kp) * 2 >= lim || ((Mp - 1) * ldc + Np) * 2 >= lim) return false;
    PlaneGemmParams p;
    std::memset(&p, 0, sizeof p);
    p.A = A;
    p.B = B;
    p.C = C;
    p.a_bytes = (uint32_t)(((M - 1) * lda + K) * 2);
    p.b_bytes = (uint32_t)((b_kn ? (K - 1) * ldb + N : (N - 1) * ldb + K) * 2);
    p.c_bytes = (uint32_t)(((M - 1) * ldc + N) * 2);
    p.lda_b = (uint32_t)(lda * 2);
    p.ldb_b = (uint32_t)(ldb * 2);
    p.ldc_b = (uint32_t)(ldc * 2);
    p.ny = ny;
    p.cap = ny;
    p.tail_b = (uint32_t)((K - (int64_t)(ny - 1) * 64) * 2);
    p.n_row_b = (uint32_t)(N * 2);
    p.nx = (int32_t)ceil_div(M, 256);
    p.nz = (int32_t)ceil_div(N, tn);
    p.jobs = p.nx * p.nz;
    p.panel = panel_of(p.nz, tn == 256 ? 8 : 16);
    p.units = p.jobs < kCUs ? p.jobs : kCUs;
    p.interleave = p.units & 7 ? 1 : 2; // (see plane_gemm)
    const bool bf = dtype == LCMA_BF16;
    const Launch launch = tn == 128 ? (b_kn ? (bf ? lcma_launch_ppn_bf16_kn : lcma_launch_ppn_f16_kn) : (bf ? lcma_launch_ppn_bf16 : lcma_launch_ppn_f16))
                          : b_kn    ? (bf ? lcma_launch_pp_kn_bf16 : lcma_launch_pp_kn_f16)
                                    : (bf ? lcma_launch_pg_bf16_t256_bf16 : lcma_launch_pg_f16_t256_f16);
    *err = launch(&p, stream);
    return true;
}

namespace {
// Plain product on few rows or a small C (csrc/lcma_few_rows.hpp): form and slices of K with the smallest time, priced on the same 5880 products as
// the tiles above and together with them (us; bf16).  A CU takes in the lines of its work-groups at `rate` bytes/ns, the slower by `crowd` the more CUs are
// at it and by `off_a`, `off_w` where rows do not start on lines; `first` besides for the launch, the first lines and the sum over the waves, `next` for every
// further work-group of a CU; and the operands come from beyond the L2 at `memory` TB/s, beyond 80 MB of them 100 MB take `far` more.  Slices of K: 1.3 for the second kernel, 0.47 a
// slice and 0.35 per MB of partial products.
struct FewRowsForm {
    int tile, cols, waves, deep, most, sliced; // most: work-groups per CU; sliced: K in slices
    double first, next, alone, rate, crowd, off_a, off_w, memory, far; // alone: rate with one work-group per CU
};
// (tiles of 64, three or more to a CU: the plane GEMM or a ping-pong kernel is faster, 1753 x 2000 x 7552 69 against 124 us, 2506 x 1056 x 4288 41 / 49; two
// to a CU: 64 x 128, 512 x 4096 x 4096 22.3 / 29.5, 320 x 4096 x 4096 19.3 / 28; tiles of 16 with eight waves and four lines in flight each fill the LDS of a CU: no
// second work-group beside the first, and slower where there is one: 1 x 14336 x 1024 12.1 us, 7.6 with the smaller form, 16 x 8192 x 512 6.0
// / 3.9; with few of them and a long K, from memory, the faster ones, 1 x 4096 x 14336 22.5 / 25.6, with a short one not, 1 x 1000 x 2048 4.3 / 3.7)
const FewRowsForm kFewRowsForms[] = {{16, 16, 4, 0, 4, 0, 1.91, 0.0, 114.0, 167.0, 0.418, 0.228, 0.139, 22.2, 7.83}, {16, 16, 8, 1, 1, 0, 3.29, 0.0, 221.0, 0.0, 1.57, 0.608, 0.304, 87.7, 3.17},
                                       {32, 32, 4, 0, 4, 0, 1.98, 0.631, 114.0, 139.0, 0.408, 0.21, 0.239, 44.9, 15.1}, {64, 64, 4, 0, 1, 0, 4.31, 0.0, 110.0, 0.0, 0.136, 0.22, 0.137, 90.0, 8.68},
                                       {64, 64, 4, 0, 1, 1, 2.96, 0.0, 121.0, 0.0, 0.298, 0.333, 0.167, 40.5, 11.3}, {64, 128, 2, 1, 1, 0, 0.0, 0.0, 1.0, 0.0, 0.0, 0.0, 0.0, 1.0, 0.0}};
const int64_t kFewRows = 1024; // (with more the 64 x 128 tiles are the plane GEMM's)
struct FewRowsPlan {
    int tile, cols, deep;
    int64_t row_blocks, col_blocks, slices, slice_steps;
    double us;
};
FewRowsPlan few_rows_plan(int64_t M, int64_t N, int64_t K, const Operands &o, int64_t scratch_bytes) {
    FewRowsPlan best{};
    for (const FewRowsForm &f : kFewRowsForms) {
        const int64_t rb = ceil_div(M, f.tile), cb = ceil_div(N, f.cols), steps = K / 32, batch = 2 * f.waves; // (steps of 32; a line of every wave)
        if (rb * cb > (int64_t)f.most * kCUs || (f.cols == 128 && M > kFewRows)) continue;
        const int64_t want = f.sliced ? kCUs / (rb * cb) : 1, slice_steps = ceil_div(ceil_div(steps, want), batch) * batch, slices = ceil_div(steps, slice_steps);
        if (f.sliced && slices < 2) continue;
        const int64_t scratch = slices > 1 ? slices * rb * f.tile * cb * f.cols * 4 : 0;
        if (scratch > scratch_bytes) continue;
        const int64_t groups = rb * cb * slices, per_cu = ceil_div(groups, kCUs), lines = std::min(slice_steps, steps) / 2;
        double us;
        if (f.cols == 128) {
            us = rounds_us(kPlain[KPAIR_64], groups, kCUs, (lines + 1) & ~(int64_t)1, o);
        } else {
            const double share = std::min(1.0, (double)groups / kCUs), line = off_lines(o, f.off_a, f.off_w) * (1.0 + f.crowd * share * share);
            us = f.first + f.next * (double)(per_cu - 1) + line * (double)(per_cu * lines * 128 * (f.tile + f.cols)) / (1e3 * (per_cu > 1 ? f.rate : f.alone)) + o.mbytes / f.memory + f.far * 0.01 * o.far();
        }
        if (slices > 1) us += 1.3 + 0.469 * (double)slices + 0.35e-6 * (double)scratch;
        if (!best.tile || us < best.us) best = FewRowsPlan{f.tile, f.cols, f.deep, rb, cb, slices, slice_steps, us};
    }
    return best;
}
} // namespace

namespace {
// The plain product on few tiles (csrc/lcma_small_plain.hip): microseconds of a form that splits K between waves, and of the fastest of the generated and
// the ping-pong kernels with N x K weights.  Both from sizes and the alignment of A's rows alone, so that either layout of B makes the
// same choice (they add the same terms in the same order: the same bits).  All measured: 470 products of 192 to 8192 rows and columns, K 192 to 14336,
// rows on lines and off, fitted to 4 to 14 % (the forms) and 14 to 20 % (what they are compared with, hence the margin).  With it the choice
// takes, K x N, 16 bit, 0.61 of the time of before in the geometric mean (every time the faster form: 0.59), fp32 0.71 (0.70), none slower; N x K
// 0.72 (0.70) and 0.75 (0.74), the worst 1.07 (920 x 632 x 616: 6.3 us).  K x N, us: 335 x 1328 x 4344 bf16 55 / 17, 448 x 312 x 3416 fp16 32 / 8, 1117
// x 608 x 7448 92 / 32, 1767 x 1216 x 10968 142 / 79, fp32 205 x 328 x 4256 96 / 23, 883 x 800 x 13800 316 / 192.
struct SmallForm {
    int tm, tn, slots;
    double start, step, crowd, off, more; // a step of 128 bytes of K, `crowd` times the share of the work-groups that fit more; `more`: a round
};
const SmallForm kSmall16[] = {{32, 32, 256, 2.56, 0.110, 0.0045, 0.104, 0.48}, {64, 64, 256, 4.07, 0.193, 0.021, 0.167, 2.97}, {64, 128, 256, 1.09, 0.264, 0.073, 0.227, 2.05}, {128, 128, 256, 0.93, 0.335, 0.134, 0.249, 2.93}};
const SmallForm kSmall32[] = {{32, 32, 256, 3.30, 0.136, 0.0, 0.035, 0.79}}; // (64 x 64, matrix instructions of one wave after the other: never ahead)
const SmallForm kOther16[] = {{64, 64, 1024, 1.62, 0.41, 0.29, 0.19, 1.14}, {128, 128, 512, 4.28, 0.90, 0.08, 0.19, 3.84}, {256, 128, 256, 3.84, 0.39, 0.59, 0.19, 3.59}, {256, 256, 256, 2.96, 0.60, 0.85, 0.19, 6.86}};
const SmallForm kOther32[] = {{64, 64, 1024, 0.65, 0.45, 1.60, 0.03, 1.60}, {128, 128, 512, 0.04, 0.71, 3.11, 0.03, 2.52}};
double small_us(const SmallForm &f, int64_t M, int64_t N, int64_t lines, bool off_line, bool in_rounds) {
    const int64_t groups = ceil_div(M, f.tm) * ceil_div(N, f.tn), full = groups / f.slots, rest = groups % f.slots;
    const double line = off_line ? 1.0 + f.off : 1.0, share = (double)rest / f.slots;
    auto step = [&](double s) { return (double)lines * line * (f.step + f.crowd * s); };
    if (in_rounds) return f.start + (double)full * (step(1.0) + f.more) + (rest ? step(share) + f.more : 0.0);
    const int64_t turns = full + (rest != 0); // (four waves to a work-group, several work-groups to a CU)
    return f.start + (double)turns * step(full ? 1.0 : share) + f.more * (double)(turns - 1);
}
} // namespace

namespace {
// The form of few tiles that the plain product takes, or null where another kernel is predicted to be as fast; *us: what it takes.
const SmallForm *small_form(int64_t M, int64_t N, int64_t K, int es, bool off_line, double *us) {
    const bool wide = es == 4;
    const int64_t lines = ceil_div(K * es, 128);
    double limit = 0.0;
    for (int i = 0; i < (wide ? 2 : 4); ++i) {
        const double other = small_us(wide ? kOther32[i] : kOther16[i], M, N, lines, off_line, true);
        if (!i || other < limit) limit = other;
    }
    limit *= wide ? 0.82 : 0.85;
    const SmallForm *form = nullptr;
    for (int i = 0; i < (wide ? 1 : 4); ++i) {
        const SmallForm &f = wide ? kSmall32[i] : kSmall16[i];
        if (i < 2 && ceil_div(M, f.tm) * ceil_div(N, f.tn) > 8 * kCUs) continue;
        const double t = small_us(f, M, N, i > 1 && lines > 2 ? (lines + 1) & ~(int64_t)1 : lines, off_line, i > 1);
        if (t < limit) {
            form = &f;
            limit = t;
        }
    }
    *us = limit;
    return form;
}
} // namespace

// Microseconds of the plain product of dense matrices on the kernels for few tiles, 0 where it does not take them.
double small_plain_us(int64_t M, int64_t N, int64_t K, int dtype) {
    const int es = dtype_size(dtype);
    double us;
    return small_form(M, N, K, es, (K * es & 127) != 0, &us) ? us : 0.0;
}

// Returns false, with nothing launched, when another kernel is predicted to be as fast or padded offsets do not fit; else *err is the launch's
// HIP error.  Arguments are checked by the caller; rows are whole 16-byte vectors.
bool small_plain(bool b_kn, int64_t M, int64_t N, int64_t K, const void *A, int64_t lda, const void *B, int64_t ldb, void *C, int64_t ldc, int dtype,
                 void *stream, int *err) {
    const int es = dtype_size(dtype);
    const int64_t lines = ceil_div(K * es, 128);
    double us;
    const SmallForm *form = small_form(M, N, K, es, (lda * es & 127) != 0, &us);
    if (!form) return false;
    const int64_t lim = (int64_t)1 << 31, Mp = ceil_div(M, 128) * 128, Np = ceil_div(N, 128) * 128, Kp = lines * 128 / es;
    if (((Mp - 1) * lda + Kp) * es >= lim || (b_kn ? (Kp - 1) * ldb + Np : (Np - 1) * ldb + Kp) * es >= lim || ((Mp - 1) * ldc + Np) * es >= lim) return false;
    const int64_t rb = ceil_div(M, form->tm), cb = ceil_div(N, form->tn);
    const uint32_t a_bytes = (uint32_t)(((M - 1) * lda + K) * es), b_bytes = (uint32_t)((b_kn ? (K - 1) * ldb + N : (N - 1) * ldb + K) * es);
    const uint32_t c_bytes = (uint32_t)(((M - 1) * ldc + N) * es), tail_b = (uint32_t)(K * es - (lines - 1) * 128);
    const int type = dtype == LCMA_BF16 ? 0 : dtype == LCMA_F16 ? 1 : 2;
    if (form->tn == 128) {
        PlaneGemmParams p;
        std::memset(&p, 0, sizeof p);
        p.A = A;
        p.B = B;
        p.C = C;
        p.a_bytes = a_bytes;
        p.b_bytes = b_bytes;
        p.c_bytes = c_bytes;
        p.lda_b = (uint32_t)(lda * es);
        p.ldb_b = (uint32_t)(ldb * es);
        p.ldc_b = (uint32_t)(ldc * es);
        p.ny = (int32_t)lines;
        p.cap = lines;
        p.tail_b = tail_b;
        p.n_row_b = (uint32_t)(N * es);
        p.nx = (int32_t)rb;
        p.nz = (int32_t)cb;
        p.jobs = p.units = (int32_t)(rb * cb);
        p.panel = panel_of(p.nz, 8);
        static const Launch launch[2][2][2] = {{{lcma_launch_plain_bf16_t64x128x64_k2t, lcma_launch_plain_bf16_t64x128x64_k2}, {lcma_launch_plain_bf16_t128x128x64_k2t, lcma_launch_plain_bf16_t128x128x64_k2}},
                                               {{lcma_launch_plain_f16_t64x128x64_k2t, lcma_launch_plain_f16_t64x128x64_k2}, {lcma_launch_plain_f16_t128x128x64_k2t, lcma_launch_plain_f16_t128x128x64_k2}}};
        *err = launch[type][form->tm == 128][b_kn](&p, stream);
        return true;
    }
    FewRowsParams q;
    std::memset(&q, 0, sizeof q);
    q.A = A;
    q.W = B;
    q.C = C;
    q.a_bytes = a_bytes;
    q.w_bytes = b_bytes;
    q.c_bytes = c_bytes;
    q.lda_b = (uint32_t)(lda * es);
    q.ldw_b = (uint32_t)(ldb * es);
    q.ldc_b = (uint32_t)(ldc * es);
    q.n_row_b = (uint32_t)(N * es);
    q.steps = (int32_t)(2 * lines);
    q.row_blocks = (int32_t)rb;
    q.block_rows = form->tm;
    q.slices = 1;
    q.slice_steps = (int32_t)(2 * lines);
    q.partial_ld = (int32_t)(cb * form->tn);
    q.tail_b = tail_b;
    typedef int (*FewLaunch)(const FewRowsParams *, int, void *);
#define LCMA_SP_ROW(TYPE) {{lcma_launch_plain_##TYPE##_t32x32x64_k4t, lcma_launch_plain_##TYPE##_t32x32x64_k4}, {lcma_launch_plain_##TYPE##_t64x64x64_k4t, lcma_launch_plain_##TYPE##_t64x64x64_k4}}
    static const FewLaunch launch[3][2][2] = {LCMA_SP_ROW(bf16), LCMA_SP_ROW(f16), {{lcma_launch_plain_f32_t32x32x32_k4t, lcma_launch_plain_f32_t32x32x32_k4}, {nullptr, nullptr}}};
    *err = launch[type][form->tm == 64][b_kn](&q, (int)(rb * cb), stream);
    return true;
}

} // namespace lcma

using namespace lcma;

// Plain GEMM for weights stored N x K on the plane GEMM, with a workspace that lets it split tile-products between
// work-groups (see include/lcma.h).
extern "C" lcma_status lcma_gemm_nt_ws(int64_t M, int64_t N, int64_t K, const void *A, int64_t lda, const void *W, int64_t ldw,
                                       void *C, int64_t ldc, lcma_dtype dtype, void *workspace, int64_t workspace_bytes,
                                       void *stream) {
    const char *who = "lcma_gemm_nt_ws";
    if (dtype != LCMA_BF16 && dtype != LCMA_F16) {
        if (!dtype_size(dtype)) return fail(LCMA_ERR_DTYPE, "%s: unknown dtype %d", who, (int)dtype);
        return lcma_gemm_nt(M, N, K, A, lda, W, ldw, C, ldc, dtype, nullptr, stream);
    }
    if (M < 0 || N < 0 || K < 0) return fail(LCMA_ERR_ARG, "%s: negative size", who);
    if (M == 0 || N == 0) return LCMA_OK;
    if (K == 0 || K % 64) return lcma_gemm_nt(M, N, K, A, lda, W, ldw, C, ldc, dtype, nullptr, stream); // steps of 64 elements
    if (!A || !W || !C) return fail(LCMA_ERR_ARG, "%s: null matrix pointer", who);
    if (lda < K || ldw < K || ldc < N) return fail(LCMA_ERR_ARG, "%s: leading dimension smaller than the row", who);
    if ((((uintptr_t)A | (uintptr_t)W | (uintptr_t)C) & 15) || (((lda | ldw | ldc) * 2) & 15))
        return fail(LCMA_ERR_ARG, "%s: pointers and leading dimensions must be multiples of 16 bytes", who);
    if (N % 8) return fail(LCMA_ERR_SHAPE, "%s: N = %lld must be a multiple of 8", who, (long long)N);
    const int64_t lim = (int64_t)1 << 31, Mp = (M + 255) / 256 * 256, Np = (N + 255) / 256 * 256;
    if (((Mp - 1) * lda + K) * 2 >= lim || ((Np - 1) * ldw + K) * 2 >= lim || ((Mp - 1) * ldc + Np) * 2 >= lim)
        return fail(LCMA_ERR_SHAPE, "%s: a matrix spans 2 GiB or more", who);
    PlaneGemmParams p;
    std::memset(&p, 0, sizeof p);
    p.A = A;
    p.B = W;
    p.C = C;
    p.a_bytes = (uint32_t)(((M - 1) * lda + K) * 2);
    p.b_bytes = (uint32_t)(((N - 1) * ldw + K) * 2);
    p.c_bytes = (uint32_t)(((M - 1) * ldc + N) * 2);
    p.lda_b = (uint32_t)(lda * 2);
    p.ldb_b = (uint32_t)(ldw * 2);
    p.ldc_b = (uint32_t)(ldc * 2);
    p.ny = (int32_t)(K / 64);
    p.n_row_b = (uint32_t)(N * 2);
    if (workspace && ((uintptr_t)workspace & 255)) return fail(LCMA_ERR_ARG, "%s: the workspace must be 256-byte aligned", who);
    const int kind = dtype == LCMA_BF16 ? PG_BF16 : PG_F16_OUT;
    const int64_t scratch = workspace ? workspace_bytes : 0;
    int t = 0, sc = 0;
    if (!tuning_schedule()) { // (a forced schedule is one of the plane GEMM's)
        // (slices only with the bytes that the interface names: half of them serve the ranges on 128 x 128 tiles, fewer are left alone)
        const Operands o = plain_operands(M, N, K, lda, ldw);
        const FewRowsPlan f = few_rows_plan(M, N, K, o, scratch >= plane_gemm_scratch_bytes(256) ? scratch : 0);
        const double planes_us = choose(kind, 1, M, N, p.ny, 0, 0, o, M > kFewRows, scratch, &t, &sc);
        int err = 0;
        const bool few = f.tile && f.us < planes_us;
        if (rounds_us(kPlain[NARROW], ceil_div(M, 256) * ceil_div(N, 128), kCUs, (p.ny + 1) & ~1, o) < (few ? f.us : planes_us) &&
            plain_product(false, M, N, K, A, lda, W, ldw, C, ldc, dtype, 0.0, stream, &err, 128))
            return err ? fail(LCMA_ERR_HIP, "%s: launch failed with HIP error %d", who, err) : LCMA_OK;
        if (few) {
            FewRowsParams q;
            std::memset(&q, 0, sizeof q);
            q.A = A;
            q.W = W;
            q.C = C;
            q.a_bytes = p.a_bytes;
            q.w_bytes = p.b_bytes;
            q.c_bytes = p.c_bytes;
            q.lda_b = p.lda_b;
            q.ldw_b = p.ldb_b;
            q.ldc_b = p.ldc_b;
            q.n_row_b = p.n_row_b;
            q.steps = (int32_t)(K / 32);
            q.row_blocks = (int32_t)f.row_blocks;
            q.block_rows = f.tile;
            q.slices = (int32_t)f.slices;
            q.slice_steps = (int32_t)f.slice_steps;
            q.partial_ld = (int32_t)(f.col_blocks * f.cols);
            q.partial = workspace;
            q.deep = f.deep;
            q.panel = panel_of((int)f.col_blocks, 8);
            const bool bf = dtype == LCMA_BF16;
            const auto launch = f.tile == 16   ? (bf ? lcma_launch_few_rows_bf16_16 : lcma_launch_few_rows_f16_16)
                                : f.tile == 32 ? (bf ? lcma_launch_few_rows_bf16_32 : lcma_launch_few_rows_f16_32)
                                               : (bf ? lcma_launch_few_rows_bf16_64 : lcma_launch_few_rows_f16_64);
            err = launch(&q, (int)(f.row_blocks * f.col_blocks * f.slices), stream);
            if (!err && f.slices > 1) err = (bf ? lcma_launch_few_rows_sum_bf16 : lcma_launch_few_rows_sum_f16)(&q, (int)M, stream);
            if (err) return fail(LCMA_ERR_HIP, "%s: launch failed with HIP error %d", who, err);
            return LCMA_OK;
        }
    }
    return plane_gemm(who, kind, p, 1, M, N, t, sc, workspace, scratch, stream);
}
