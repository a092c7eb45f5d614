// Instances of the plane GEMM (csrc/lcma_plane_gemm.hpp) and of its fix-up kernel.
#include "lcma_kpair.hpp"
#include "lcma_pingpong_narrow.hpp"

using namespace lcma;

#define LCMA_PERSISTENT(NAME, KIND, OUT)                                                                               \
    extern "C" __global__ __launch_bounds__(512, 2) void lcma_k_pg_pp_##NAME(const lcma::PlaneGemmParams) {           \
        using G = PingPongGemm<KIND, OUT>;                                                                             \
        __shared__ __attribute__((aligned(16))) char smem[G::LDS_BYTES];                                               \
        G::run((LCMA_LDS char *)smem);                                                                                 \
    }
#define LCMA_LAUNCH_PERSISTENT(NAME)                                                                                   \
    if (p->interleave) {                                                                                               \
        lcma_k_pg_pp_##NAME<<<dim3(p->units), dim3(512), 0, (hipStream_t)stream>>>(*p);                                \
        return (int)hipGetLastError();                                                                                 \
    }

#define LCMA_PLANE_GEMM(NAME, KIND, TM, TN, WGM, WGN, OCC, OUT)                                                        \
    extern "C" __global__ __launch_bounds__(64 * WGM * WGN, OCC) void lcma_k_pg_##NAME(const lcma::PlaneGemmParams p) { \
        using G = PlaneGemm<KIND, TM, TN, WGM, WGN, OUT, false>;                                                       \
        __shared__ __attribute__((aligned(16))) char smem[G::LDS_BYTES];                                               \
        G::run(p, (LCMA_LDS char *)smem);                                                                              \
    }                                                                                                                  \
    extern "C" __global__ __launch_bounds__(64 * WGM * WGN, OCC) void lcma_k_pg_split_##NAME(const lcma::PlaneGemmParams p) { \
        using G = PlaneGemm<KIND, TM, TN, WGM, WGN, OUT, true>;                                                        \
        __shared__ __attribute__((aligned(16))) char smem[G::LDS_BYTES];                                               \
        G::run(p, (LCMA_LDS char *)smem);                                                                              \
    }                                                                                                                  \
    extern "C" __global__ __launch_bounds__(64 * WGM * WGN) void lcma_k_pg_fixup_##NAME(const lcma::PlaneGemmParams p) { \
        using G = PlaneGemm<KIND, TM, TN, WGM, WGN, OUT, true>;                                                        \
        __shared__ __attribute__((aligned(16))) char smem[G::LDS_BYTES];                                               \
        G::fixup(p, (LCMA_LDS char *)smem);                                                                            \
    }                                                                                                                  \
    LCMA_PERSISTENT(NAME, KIND, OUT)                                                                                  \
    /* whole tile-products in turn: the ping-pong kernel on the large tile; one tile-product per work-group when cap is a whole tile-product and there are as many work-groups as              \
       tile-products, else the persistent kernel and the kernel that adds the pieces */                                  \
    extern "C" int lcma_launch_pg_##NAME(const lcma::PlaneGemmParams *p, void *stream) {                               \
        LCMA_LAUNCH_PERSISTENT(NAME)                                                                                  \
        if (p->cap == p->ny && p->units == p->jobs) {                                                                  \
            lcma_k_pg_##NAME<<<dim3(p->units), dim3(64 * WGM * WGN), 0, (hipStream_t)stream>>>(*p);                    \
            return (int)hipGetLastError();                                                                             \
        }                                                                                                              \
        lcma_k_pg_split_##NAME<<<dim3(p->units), dim3(64 * WGM * WGN), 0, (hipStream_t)stream>>>(*p);                  \
        if (const hipError_t e = hipGetLastError()) return (int)e;                                                     \
        if (p->cap % p->ny && p->units > 1)                                                                            \
            lcma_k_pg_fixup_##NAME<<<dim3(p->units - 1), dim3(64 * WGM * WGN), 0, (hipStream_t)stream>>>(*p);          \
        return (int)hipGetLastError();                                                                                 \
    }

#define LCMA_KPAIR_KERNEL(NAME, KIND, TM, OUT, RUN)                                                                    \
    extern "C" __global__ __launch_bounds__(512, 2) void lcma_k_##NAME(const lcma::PlaneGemmParams p) {                \
        using G = KPair<KIND, OUT, TM>;                                                                                  \
        __shared__ __attribute__((aligned(16))) char smem[G::LDS_BYTES];                                               \
        G::RUN(p, (LCMA_LDS char *)smem);                                                                              \
    }
#define LCMA_KPAIR(NAME, KIND, OUT)                                                                                    \
    extern "C" __global__ __launch_bounds__(256, 2) void lcma_k_pg_two_##NAME(const lcma::PlaneGemmParams p) {         \
        using G = PlaneGemm<KIND, 128, 128, 2, 2, OUT, false>;                                                         \
        __shared__ __attribute__((aligned(16))) char smem[G::LDS_BYTES];                                               \
        G::run(p, (LCMA_LDS char *)smem);                                                                              \
    }                                                                                                                  \
    LCMA_KPAIR_KERNEL(pg_##NAME, KIND, 128, OUT, run)                                                                   \
    LCMA_KPAIR_KERNEL(pg_low_##NAME, KIND, 64, OUT, run)                                                               \
    LCMA_KPAIR_KERNEL(pg_ranges_##NAME, KIND, 128, OUT, run_ranges)                                                     \
    LCMA_KPAIR_KERNEL(pg_fixup_##NAME, KIND, 128, OUT, fixup)                                                           \
    /* whole tile-products, a work-group each (also where they are to be dealt in turn); slices of K, which the caller adds; ranges of steps, \
       dealt to 512 work-groups: of this kernel 256 run at a time */                                                   \
    extern "C" int lcma_launch_pg_##NAME(const lcma::PlaneGemmParams *p, void *stream) {                               \
        if (p->interleave == 3) return LCMA_KPAIR_SLICES_##KIND(p, stream);                                            \
        if (p->interleave == 4) { /* two work-groups to a CU */                                                        \
            lcma_k_pg_two_##NAME<<<dim3(p->jobs), dim3(256), 0, (hipStream_t)stream>>>(*p);                            \
            return (int)hipGetLastError();                                                                             \
        }                                                                                                              \
        if (p->interleave == 5) { /* tiles of 64 x 128 */                                                              \
            lcma_k_pg_low_##NAME<<<dim3(p->jobs), dim3(512), 0, (hipStream_t)stream>>>(*p);                            \
            return (int)hipGetLastError();                                                                             \
        }                                                                                                              \
        if (!p->partial) {                                                                                             \
            lcma_k_pg_##NAME<<<dim3(p->jobs), dim3(512), 0, (hipStream_t)stream>>>(*p);                                \
            return (int)hipGetLastError();                                                                             \
        }                                                                                                              \
        lcma::PlaneGemmParams q = *p;                                                                                  \
        q.cap *= 2;                                                                                                    \
        q.units = (q.units + 1) / 2;                                                                                   \
        lcma_k_pg_ranges_##NAME<<<dim3(q.units), dim3(512), 0, (hipStream_t)stream>>>(q);                              \
        if (const hipError_t e = hipGetLastError()) return (int)e;                                                     \
        if (q.cap % q.ny && q.units > 1) lcma_k_pg_fixup_##NAME<<<dim3(q.units - 1), dim3(512), 0, (hipStream_t)stream>>>(q); \
        return (int)hipGetLastError();                                                                                 \
    }
#define LCMA_KPAIR_SLICES(NAME, KIND)                                                                                  \
    LCMA_KPAIR_KERNEL(pg_slices_##NAME, KIND, 128, F32, run_slices)                                                     \
    static int launch_slices_##NAME(const lcma::PlaneGemmParams *p, void *stream) {                                    \
        lcma_k_pg_slices_##NAME<<<dim3(p->units / 2), dim3(512), 0, (hipStream_t)stream>>>(*p);                            \
        return (int)hipGetLastError();                                                                                 \
    }
LCMA_KPAIR_SLICES(bf16, BF16)
LCMA_KPAIR_SLICES(f16, F16)
#define LCMA_KPAIR_SLICES_BF16 launch_slices_bf16
#define LCMA_KPAIR_SLICES_F16 launch_slices_f16
#define LCMA_KPAIR_SLICES_FP8(P, STREAM) (int)hipErrorInvalidValue /* (FP8 products have no scratch for slices) */

// name: operand kind, tile, type of C
LCMA_PLANE_GEMM(fp8_t256_bf16, FP8, 256, 256, 2, 4, 1, BF16)
LCMA_KPAIR(fp8_t128_bf16, FP8, BF16)
LCMA_PLANE_GEMM(fp8_t256_f16, FP8, 256, 256, 2, 4, 1, F16)
LCMA_KPAIR(fp8_t128_f16, FP8, F16)
LCMA_PLANE_GEMM(f16_t256_f16, F16, 256, 256, 2, 4, 1, F16)
LCMA_KPAIR(f16_t128_f16, F16, F16)
LCMA_PLANE_GEMM(f16_t256_f32, F16, 256, 256, 2, 4, 1, F32)
LCMA_KPAIR(f16_t128_f32, F16, F32)
LCMA_PLANE_GEMM(bf16_t256_bf16, BF16, 256, 256, 2, 4, 1, BF16)
LCMA_KPAIR(bf16_t128_bf16, BF16, BF16)



// The ping-pong kernels of the plain product (csrc/plane_gemm.cc, plain_product): K x N operand on the 256 x 256 tile, either
// operand on the 256 x 128 tile.
#define LCMA_PINGPONG_KN(NAME, KIND)                                                                                   \
    extern "C" __global__ __launch_bounds__(512, 2) void lcma_k_pp_kn_##NAME(const lcma::PlaneGemmParams) {            \
        using G = PingPongGemm<KIND, KIND, true>;                                                                      \
        __shared__ __attribute__((aligned(16))) char smem[G::LDS_BYTES];                                               \
        G::run((LCMA_LDS char *)smem);                                                                                 \
    }                                                                                                                  \
    extern "C" int lcma_launch_pp_kn_##NAME(const lcma::PlaneGemmParams *p, void *stream) {                            \
        lcma_k_pp_kn_##NAME<<<dim3(p->units), dim3(512), 0, (hipStream_t)stream>>>(*p);                                \
        return (int)hipGetLastError();                                                                                 \
    }
#define LCMA_PINGPONG_NARROW(NAME, KIND, KN)                                                                           \
    extern "C" __global__ __launch_bounds__(512, 2) void lcma_k_ppn_##NAME(const lcma::PlaneGemmParams p) {            \
        using G = PingPongNarrow<KIND, KIND, KN>;                                                                      \
        __shared__ __attribute__((aligned(16))) char smem[G::LDS_BYTES];                                               \
        G::run(p, (LCMA_LDS char *)smem);                                                                              \
    }                                                                                                                  \
    extern "C" int lcma_launch_ppn_##NAME(const lcma::PlaneGemmParams *p, void *stream) {                              \
        lcma_k_ppn_##NAME<<<dim3(p->jobs), dim3(512), 0, (hipStream_t)stream>>>(*p);                                   \
        return (int)hipGetLastError();                                                                                 \
    }
LCMA_PINGPONG_KN(bf16, BF16)
LCMA_PINGPONG_KN(f16, F16)
LCMA_PINGPONG_NARROW(bf16, BF16, false)
LCMA_PINGPONG_NARROW(f16, F16, false)
LCMA_PINGPONG_NARROW(bf16_kn, BF16, true)
LCMA_PINGPONG_NARROW(f16_kn, F16, true)
