// Instances of the plane GEMM (csrc/lcma_plane_gemm.hpp) and of its fix-up kernel.
#include "lcma_pingpong_narrow.hpp"

using namespace lcma;

// on the 128 x 128 tile the kernel of the Split-Group ranges also runs whole tile-products in turn
#define LCMA_PERSISTENT_128(NAME, KIND, OUT)
#define LCMA_LAUNCH_PERSISTENT_128(NAME)
#define LCMA_PERSISTENT_256(NAME, KIND, OUT)                                                                           \
    extern "C" __global__ __launch_bounds__(512, 2) void lcma_k_pg_pp_##NAME(const lcma::PlaneGemmParams) {           \
        using G = PingPongGemm<KIND, OUT>;                                                                             \
        __shared__ __attribute__((aligned(16))) char smem[G::LDS_BYTES];                                               \
        G::run((LCMA_LDS char *)smem);                                                                                 \
    }
#define LCMA_LAUNCH_PERSISTENT_256(NAME)                                                                               \
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
    LCMA_PERSISTENT_##TM(NAME, KIND, OUT)                                                                              \
    /* whole tile-products in turn: the ping-pong kernel on the large tile; one tile-product per work-group when cap is a whole tile-product and there are as many work-groups as              \
       tile-products, else the persistent kernel and the kernel that adds the pieces */                                  \
    extern "C" int lcma_launch_pg_##NAME(const lcma::PlaneGemmParams *p, void *stream) {                               \
        LCMA_LAUNCH_PERSISTENT_##TM(NAME)                                                                              \
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

// name: operand kind, tile, type of C
LCMA_PLANE_GEMM(fp8_t256_bf16, FP8, 256, 256, 2, 4, 1, BF16)
LCMA_PLANE_GEMM(fp8_t128_bf16, FP8, 128, 128, 2, 2, 2, BF16)
LCMA_PLANE_GEMM(fp8_t256_f16, FP8, 256, 256, 2, 4, 1, F16)
LCMA_PLANE_GEMM(fp8_t128_f16, FP8, 128, 128, 2, 2, 2, F16)
LCMA_PLANE_GEMM(f16_t256_f16, F16, 256, 256, 2, 4, 1, F16)
LCMA_PLANE_GEMM(f16_t128_f16, F16, 128, 128, 2, 2, 2, F16)
LCMA_PLANE_GEMM(f16_t256_f32, F16, 256, 256, 2, 4, 1, F32)
LCMA_PLANE_GEMM(f16_t128_f32, F16, 128, 128, 2, 2, 2, F32)
LCMA_PLANE_GEMM(bf16_t256_bf16, BF16, 256, 256, 2, 4, 1, BF16)
LCMA_PLANE_GEMM(bf16_t128_bf16, BF16, 128, 128, 2, 2, 2, BF16)



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
