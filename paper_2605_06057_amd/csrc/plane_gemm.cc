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

namespace lcma {

namespace {
const int kCUs = 256;
typedef int (*Launch)(const PlaneGemmParams *, void *);
Launch launcher(int kind, int tile) {
    switch (kind * 2 + (tile == 256)) {
    case PG_FP8_BF16 * 2 + 1: return lcma_launch_pg_fp8_t256_bf16;
    case PG_FP8_BF16 * 2: return lcma_launch_pg_fp8_t128_bf16;
    case PG_FP8_F16 * 2 + 1: return lcma_launch_pg_fp8_t256_f16;
    case PG_FP8_F16 * 2: return lcma_launch_pg_fp8_t128_f16;
    case PG_F16 * 2 + 1: return lcma_launch_pg_f16_t256_f16;
    case PG_F16 * 2: return lcma_launch_pg_f16_t128_f16;
    case PG_BF16 * 2 + 1: return lcma_launch_pg_bf16_t256_bf16;
    case PG_BF16 * 2: return lcma_launch_pg_bf16_t128_bf16;
    case PG_F16_OUT * 2 + 1: return lcma_launch_pg_f16_t256_f16;
    case PG_F16_OUT * 2: return lcma_launch_pg_f16_t128_f16;
    case PG_F16_F32 * 2 + 1: return lcma_launch_pg_f16_t256_f32;
    case PG_F16_F32 * 2: return lcma_launch_pg_f16_t128_f32;
    }
    return nullptr;
}
int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
// work-groups that run at one time: one 256 x 256 tile (128 KB of LDS) or two 128 x 128 tiles (64 KB each) per CU
int slots_of(int tile) { return tile == 256 ? kCUs : 2 * kCUs; }
} // namespace

int64_t plane_gemm_scratch_bytes(int tile) { return (int64_t)slots_of(tile) * 2 * tile * tile * 4; }

namespace {
// Tile and schedule together, by the time the slowest work-group takes.  All constants are measured (us; random operands;
// f: share of the chip's work-group slots that a round fills: with fewer work-groups the memory side answers sooner and
// the clock is higher).
//   256 x 256, whole tile-products in turn (ping-pong kernel, csrc/lcma_pingpong.hpp): a step of 128 bytes of K takes 1.52
//     with all 256 work-groups (8192 x 14336 x 4096: 712 us in 7 rounds of 64 steps; 7 planes of 4096 x 7168 x 2048: 724 us),
//     1.16 with 128 (2048 x 4096 x 4096: 81 us), 0.98 with 64 (2048 x 2048 x 7168: 110 us); a tile-product 6 besides (12
//     with fp32 output), and the start of the pipeline 1.5;
//   256 x 256, one work-group per tile-product (PlaneGemm): 1.62 (FP8: 2.05) a step, but a shorter start: the faster one
//     up to about eight steps (4096 x 4096 x 128: 11.0 against 11.8 us, x 256: 15.4 against 15.7, x 512: 22.4 both);
//   128 x 128, two work-groups per CU: 1.06 a step of both (FP8: 1.16) with 512 work-groups, 0.72 to 0.9 with 256, 0.62
//     with a few (2048 x 4096 x 4096: 68 us; 1024 x 4096 x 4096: 48 us; x 16384: 232 us; 64 x 4096 x 4096: 41 us): the one to take when the large
//     tiles leave much of the chip idle;
//   Split-Group ranges: 1.75 (1.6; FP8 2.0 and 1.1) a step, 6 (3) a tile-product and 65 (20, and 0.45 for every piece of a tile; FP8 40)
//     for the pieces: nearly every work-group holds two, 134 (67) MB of fp32 partial sums in all, written at the end of the first
//     kernel and read back by the second (1024 x 4096 x 16384: 161 us against 232 with 128 x 128 tiles; 512 x 4096 x 14336: 95 against 221): few
//     tile-products and a long K only (2463 x 8344 x 6528: 334 against 248 with the ping-pong kernel; neighbouring tiles of the 128 x
//     128 form start at different k and share little in L2: 857 x 3720 x 7040 112 against 91 with a work-group per tile).
// tile, schedule: 0 = choose.  Returns microseconds (0 when nothing fits).
double choose(int kind, int planes, int64_t rows, int64_t cols, int ny, int tile, int schedule, int64_t scratch_bytes, int *best_tile,
              int *best_sched) {
    const bool fp8 = kind == PG_FP8_BF16 || kind == PG_FP8_F16;
    const double out = kind == PG_F16_F32 ? 2.0 : 1.0; // a tile of fp32 takes twice as long to write
    double best = 0.0;
    *best_tile = *best_sched = 0;
    for (int t : {256, 128}) {
        if (tile && t != tile) continue;
        const int64_t jobs = (int64_t)planes * ceil_div(rows, t) * ceil_div(cols, t), slots = slots_of(t);
        for (int sc : {1, 2, 3}) {
            if (schedule && sc != schedule) continue;
            const bool pingpong = t == 256 && sc == 3;
            // (the 128 x 128 FP8 kernel loses with whole tile-products in turn: it does not fetch the next scales ahead)
            if (!schedule && sc == 3 && fp8 && t == 128) continue;
            // planes lie back to back: only the ping-pong kernel lets a tile hang over the end of one
            if (planes > 1 && !pingpong && (rows % t || cols % t)) continue;
            if (sc == 2 && scratch_bytes < plane_gemm_scratch_bytes(t)) continue;
            double cost;
            if (sc == 2) {
                const double cap = (double)ceil_div(jobs * ny, slots), pieces = t == 256 ? 65.0 : fp8 ? 40.0 : 20.0 + 0.45 * (double)ny / cap;
                cost = cap * (t == 256 ? fp8 ? 2.0 : 1.75 : fp8 ? 1.1 : 1.6) + (t == 256 ? 6.0 : 3.0) * out * (double)jobs / (double)slots + pieces;
            } else {
                const int64_t full = jobs / slots, rest = jobs % slots;
                auto round = [&](double f) {
                    if (pingpong) return (double)((ny + 1) & ~1) * (0.80 + 0.72 * f) + 6.0 * out;
                    if (t == 256) return (double)ny * (fp8 ? 1.0 + 1.05 * f : 0.85 + 0.77 * f) + 6.0 * out;
                    const double alone = 0.62 + 0.5 * (f < 0.5 ? f : 0.5); // one work-group per CU up to f = 0.5
                    return (double)ny * (alone + (f > 0.5 ? 0.5 * (f - 0.5) : 0.0)) + (sc == 3 && full ? 2.5 : 3.0) * out;
                };
                cost = (double)full * round(1.0) + (rest ? round((double)rest / (double)slots) : 0.0) + (pingpong ? 1.5 : 0.0);
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
// lcma_select_dataflow: measured 54.6 us at 53 predicted (7 planes, 2048 x 4096 x 4096), 318 / 315 (6144^3), 695 / 695 (FFN).
double batched_plane_gemm_seconds(bool fp32_out, int planes, int64_t rows, int64_t cols, int ny) {
    int t = 0, sc = 0;
    const double us = choose(fp32_out ? PG_F16_F32 : PG_F16, planes, rows, cols, ny, 0, tuning_schedule(), 0, &t, &sc);
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
// (padded sizes; when batched only the ping-pong kernel takes planes that are no whole tiles).  tile: 256 or 128, 0 = choose.
// schedule: 0 = choose, 1 = one tile-product per work-group, 2 = Split-Group ranges (needs `scratch` of
// plane_gemm_scratch_bytes(tile) bytes), 3 = persistent work-groups that each take every units-th whole tile-product.
lcma_status plane_gemm(const char *who, int kind, PlaneGemmParams p, int planes, int64_t rows, int64_t cols, int tile,
                       int schedule, void *scratch, int64_t scratch_bytes, void *stream) {
    const int forced = tuning_schedule();
    if (forced) schedule = forced;
    int best_tile = 0, best_sched = 0;
    choose(kind, planes, rows, cols, p.ny, tile, schedule, scratch ? scratch_bytes : 0, &best_tile, &best_sched);
    if (!best_tile) {
        if (schedule == 2)
            return fail(LCMA_ERR_ARG, "%s: the Split-Group schedule needs %lld bytes of scratch", who,
                        (long long)plane_gemm_scratch_bytes(tile ? tile : 256));
        return fail(LCMA_ERR_SHAPE, "%s: planes must be whole tiles", who);
    }
    tile = best_tile;
    schedule = best_sched;
    Launch launch = launcher(kind, tile);
    if (!launch) return fail(LCMA_ERR_NOKERNEL, "%s: no plane GEMM kernel of kind %d", who, kind);
    if (!p.tail_b) p.tail_b = 128; // whole steps
    p.nx = (int32_t)ceil_div(rows, tile);
    p.nz = (int32_t)ceil_div(cols, tile);
    const int64_t jobs = (int64_t)planes * p.nx * p.nz, total = jobs * p.ny;
    if (total >= ((int64_t)1 << 31)) return fail(LCMA_ERR_SHAPE, "%s: too many tile steps", who);
    p.jobs = (int32_t)jobs;
    p.panel = panel_of(p.nz, 8);
    const int slots = slots_of(tile);
    p.interleave = 0;
    if (schedule == 3) { // persistent work-groups, whole tile-products u, u + units, ...
        p.units = (int32_t)(jobs < slots ? jobs : slots);
        p.cap = p.ny;
        // batches of planes: rounds of consecutive tile-products; one product: an eighth of them per XCD (see
        // PlaneGemm::run), which needs the same number of work-groups on every XCD
        p.interleave = planes > 1 || (p.units & 7) ? 1 : 2;
        p.partial = nullptr;
    } else if (schedule == 2) {
        p.units = (int32_t)(total < slots ? total : slots);
        p.cap = ceil_div(total, p.units);
        p.units = (int32_t)ceil_div(total, p.cap); // no idle work-group at the end
        p.partial = scratch;
    } else {
        p.units = (int32_t)jobs;
        p.cap = p.ny;
        p.partial = nullptr;
    }
    if (const int err = launch(&p, stream)) return fail(LCMA_ERR_HIP, "%s: plane GEMM launch failed with HIP error %d", who, err);
    return LCMA_OK;
}

// Microseconds of the plain product on the ping-pong kernel with tiles of 256 x tn (f as in choose()).  256 x 128: 0.52 + 0.38 f a
// step (K x N: 0.60 + 0.32 f, its fragments wait for their own reads) and 4 a round (K x N: 2048 x 4096 x 4096 62 against 87 for
// the generated kernel, 1024 x 4096 x 4096 50 / 56, 2048 x 4096 x 14336 210 / 284, 704 x 704 x 8000 80 / 98); 256 x 256: as in
// choose() for either layout (K x N: 6144^3 394 / 495, 8192 x 14336 x 4096 704 / 863); 15 % more when rows do not start on
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
// predicted to take less than the `limit_us` given, or when padded offsets do not fit; else *err is the launch's HIP error.
bool plain_product(bool b_kn, int64_t M, int64_t N, int64_t K, const void *A, int64_t lda, const void *B, int64_t ldb, void *C, int64_t ldc,
                   int dtype, double limit_us, void *stream, int *err) {
    const int ny = (int)ceil_div(K, 64);
    auto cost = [&](int tn) { return plain_product_us(b_kn, tn, M, N, K, lda % 64 || ldb % 64); };
    const int tn = cost(256) < cost(128) ? 256 : 128;
    if (cost(tn) >= limit_us) return false;
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
// Plain product on few rows or a small C (csrc/lcma_few_rows.hpp): form and slices of K with the smallest time, all constants measured (us;
// bf16, three sets of operands in turn).  A CU takes in the lines of its work-groups at `rate` bytes/ns; `first` besides for the launch, the
// first lines and the sum over the waves, `next` for every further work-group of a CU; and what the operands themselves take from
// beyond the L2, as far as it does not lie behind the lines, 8 TB/s.  Slices of K: 1.3 for the second kernel, 0.25 a slice and 0.35 per MB of
// partial products.  At 190 shapes, M 1 to 8872, N 8 to 14336, K 128 to 14400, with the workspace and without, the choice takes 1.009 of the time of
// the fastest form (the plane GEMM among them), at the worst 1.23; the rates of the kernel before, 36 bytes/ns for all tiles: 1.27 and 2.1.
struct FewRowsForm {
    int tile, waves, deep, most; // most: work-groups per CU
    double first, next, alone, rate;    // alone: rate with one work-group per CU
};
// (tiles of 64, three or more to a CU: the plane GEMM or a ping-pong kernel is faster, 1753 x 2000 x 7552 69 against 124 us, 2506 x 1056 x 4288 41 / 49;
// tiles of 16 with eight waves and four lines in flight each fill the LDS of a CU: no second work-group beside the first, and slower
// where there is one: 1 x 14336 x 1024 12.1 us, 7.6 with the smaller form, 16 x 8192 x 512 6.0 / 3.9; with few of them and a long K
// the faster ones, 1 x 4096 x 14336 22.5 / 25.6, with a short one not, 1 x 1000 x 2048 4.3 / 3.7)
const FewRowsForm kFewRowsForms[] = {{16, 4, 0, 4, 2.8, 0.3, 90.0, 100.0}, {16, 8, 1, 1, 3.5, 0.0, 115.0, 0.0}, {32, 4, 0, 4, 3.1, 0.85, 100.0, 100.0}, {64, 4, 0, 2, 4.8, 3.5, 105.0, 105.0}};
struct FewRowsPlan {
    int tile, deep;
    int64_t row_blocks, col_blocks, slices, slice_steps;
    double us;
};
FewRowsPlan few_rows_plan(int64_t M, int64_t N, int64_t K, int64_t scratch_bytes) {
    FewRowsPlan best{};
    for (const FewRowsForm &f : kFewRowsForms) {
        const int64_t rb = ceil_div(M, f.tile), cb = ceil_div(N, f.tile), steps = K / 32, batch = 2 * f.waves; // (steps of 32; a line of every wave)
        if (rb * cb > (int64_t)f.most * kCUs) continue;
        for (int64_t want : {(int64_t)1, kCUs / (rb * cb)}) {
            if (want < 1 || (want > 1 && f.tile != 64)) continue;
            const int64_t slice_steps = ceil_div(ceil_div(steps, want), batch) * batch, slices = ceil_div(steps, slice_steps);
            const int64_t scratch = slices > 1 ? slices * rb * f.tile * cb * f.tile * 4 : 0;
            if (scratch > scratch_bytes) continue;
            const int64_t per_cu = ceil_div(rb * cb * slices, kCUs), lines = std::min(slice_steps, steps) / 2;
            double us = f.first + f.next * (double)(per_cu - 1) + (double)(per_cu * lines * 256 * f.tile) / (1e3 * (per_cu > 1 ? f.rate : f.alone)) + (double)((M + N) * K * 2) / 8e6;
            if (slices > 1) us += 1.3 + 0.25 * (double)slices + 0.35e-6 * (double)scratch;
            if (!best.tile || us < best.us) best = FewRowsPlan{f.tile, f.deep, rb, cb, slices, slice_steps, us};
        }
    }
    return best;
}
} // namespace

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
    if (!tuning_schedule()) { // (a forced schedule is one of the plane GEMM's)
        // (slices only with the bytes that the interface names: half of them serve the ranges on 128 x 128 tiles, fewer are left alone)
        const FewRowsPlan f = few_rows_plan(M, N, K, scratch >= plane_gemm_scratch_bytes(256) ? scratch : 0);
        int t = 0, sc = 0;
        const double planes_us = choose(kind, 1, M, N, p.ny, 0, 0, scratch, &t, &sc);
        int err = 0;
        // (against the ranges of steps a quarter on the safe side with two tiles of 64 per CU: 512 x 4096 x 14336 92 us, priced 112, in few rows 109, priced 95;
        // 512 x 4096 x 12288 87 / 98; but 512 x 4096 x 8192 57 / 50; with fewer or smaller tiles both prices hold, 3 x 12672 x 10432 74 / 50,
        // 1 x 10440 x 13440 75 / 53)
        const bool full = f.tile == 64 && f.row_blocks * f.col_blocks > kCUs;
        const bool few = f.tile && f.us * (sc == 2 && full ? 1.25 : 1.0) < planes_us;
        // (1.5 us on the safe side: 840 x 5592 x 768 15.7 against 14.4, 4358 x 256 x 640 10.4 against 9.2)
        if (plain_product(false, M, N, K, A, lda, W, ldw, C, ldc, dtype, (few ? f.us : planes_us) - 1.5, stream, &err))
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
            q.partial_ld = (int32_t)(f.col_blocks * f.tile);
            q.partial = workspace;
            q.deep = f.deep;
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
    return plane_gemm(who, kind, p, 1, M, N, 0, 0, workspace, scratch, stream);
}
