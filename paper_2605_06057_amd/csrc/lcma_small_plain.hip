// Instances of the plain product of lcma_gemm and lcma_gemm_nt on few tiles: the waves of a work-group split K (csrc/lcma_few_rows.hpp, tiles of 32 and 64,
// and csrc/lcma_kpair.hpp).  The names say what the generated kernels' say: tile, depth of a step, parts of K, t for N x K weights.
#include "lcma_few_rows.hpp"
#include "lcma_kpair.hpp"

using namespace lcma;

#define LCMA_SMALL_PLAIN(NAME, KIND, T, KN)                                                                            \
    extern "C" __global__ __launch_bounds__(256, 1) void lcma_k_##NAME(const lcma::FewRowsParams p) {                  \
        using G = FewRows<KIND, T, 4, 2, KN, true>;                                                                    \
        __shared__ __attribute__((aligned(16))) char smem[G::LDS_BYTES];                                               \
        G::run(p, (LCMA_LDS char *)smem);                                                                              \
    }                                                                                                                  \
    extern "C" int lcma_launch_##NAME(const lcma::FewRowsParams *p, int grid, void *stream) {                          \
        lcma_k_##NAME<<<dim3(grid), dim3(256), 0, (hipStream_t)stream>>>(*p);                                          \
        return (int)hipGetLastError();                                                                                 \
    }
LCMA_SMALL_PLAIN(plain_bf16_t32x32x64_k4, BF16, 32, true)
LCMA_SMALL_PLAIN(plain_bf16_t32x32x64_k4t, BF16, 32, false)
LCMA_SMALL_PLAIN(plain_bf16_t64x64x64_k4, BF16, 64, true)
LCMA_SMALL_PLAIN(plain_bf16_t64x64x64_k4t, BF16, 64, false)
LCMA_SMALL_PLAIN(plain_f16_t32x32x64_k4, F16, 32, true)
LCMA_SMALL_PLAIN(plain_f16_t32x32x64_k4t, F16, 32, false)
LCMA_SMALL_PLAIN(plain_f16_t64x64x64_k4, F16, 64, true)
LCMA_SMALL_PLAIN(plain_f16_t64x64x64_k4t, F16, 64, false)
LCMA_SMALL_PLAIN(plain_f32_t32x32x32_k4, F32, 32, true)
LCMA_SMALL_PLAIN(plain_f32_t32x32x32_k4t, F32, 32, false)

#define LCMA_KPAIR_PLAIN(NAME, KIND, TM)                                                                               \
    extern "C" __global__ __launch_bounds__(512, 2) void lcma_k_##NAME(const lcma::PlaneGemmParams p) {                \
        using G = KPair<KIND, KIND, TM, true>;                                                                         \
        __shared__ __attribute__((aligned(16))) char smem[G::LDS_BYTES];                                               \
        G::run(p, (LCMA_LDS char *)smem);                                                                              \
    }                                                                                                                  \
    extern "C" int lcma_launch_##NAME(const lcma::PlaneGemmParams *p, void *stream) {                                  \
        lcma_k_##NAME<<<dim3(p->jobs), dim3(512), 0, (hipStream_t)stream>>>(*p);                                       \
        return (int)hipGetLastError();                                                                                 \
    }
// N x K weights: the tiles of the plane GEMM (csrc/lcma_plane_gemm.hip), dealt 0 (128 x 128) or 5 (64 x 128)
#define LCMA_KPAIR_PLAIN_T(NAME, TYPE, DEALT)                                                                          \
    extern "C" int lcma_launch_pg_##TYPE##_t128_##TYPE(const lcma::PlaneGemmParams *p, void *stream);                  \
    extern "C" int lcma_launch_##NAME(const lcma::PlaneGemmParams *p, void *stream) {                                  \
        lcma::PlaneGemmParams q = *p;                                                                                  \
        q.interleave = DEALT;                                                                                          \
        return lcma_launch_pg_##TYPE##_t128_##TYPE(&q, stream);                                                        \
    }
LCMA_KPAIR_PLAIN(plain_bf16_t128x128x64_k2, BF16, 128)
LCMA_KPAIR_PLAIN_T(plain_bf16_t128x128x64_k2t, bf16, 0)
LCMA_KPAIR_PLAIN(plain_bf16_t64x128x64_k2, BF16, 64)
LCMA_KPAIR_PLAIN_T(plain_bf16_t64x128x64_k2t, bf16, 5)
LCMA_KPAIR_PLAIN(plain_f16_t128x128x64_k2, F16, 128)
LCMA_KPAIR_PLAIN_T(plain_f16_t128x128x64_k2t, f16, 0)
LCMA_KPAIR_PLAIN(plain_f16_t64x128x64_k2, F16, 64)
LCMA_KPAIR_PLAIN_T(plain_f16_t64x128x64_k2t, f16, 5)
