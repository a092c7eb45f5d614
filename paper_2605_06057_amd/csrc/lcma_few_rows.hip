// Instances of the plain product on few rows (csrc/lcma_few_rows.hpp) and of the kernel that adds the slices of K.
#include "lcma_few_rows.hpp"

using namespace lcma;

#define LCMA_FEW_ROWS_KERNEL(NAME, KIND, T, WK, S)                                                                     \
    extern "C" __global__ __launch_bounds__(64 * WK, 1) void lcma_k_few_rows_##NAME(const lcma::FewRowsParams p) {     \
        using G = FewRows<KIND, T, WK, S>;                                                                             \
        __shared__ __attribute__((aligned(16))) char smem[G::LDS_BYTES];                                               \
        G::run(p, (LCMA_LDS char *)smem);                                                                              \
    }
#define LCMA_FEW_ROWS(NAME, KIND, T, WK, S)                                                                            \
    LCMA_FEW_ROWS_KERNEL(NAME, KIND, T, WK, S)                                                                         \
    extern "C" int lcma_launch_few_rows_##NAME(const lcma::FewRowsParams *p, int grid, void *stream) {                 \
        lcma_k_few_rows_##NAME<<<dim3(grid), dim3(64 * WK), 0, (hipStream_t)stream>>>(*p);                             \
        return (int)hipGetLastError();                                                                                 \
    }
// Tiles of 64 x 128: those of the plane GEMM (csrc/lcma_plane_gemm.hip).
extern "C" int lcma_launch_pg_f16_t128_f16(const lcma::PlaneGemmParams *p, void *stream);
extern "C" int lcma_launch_pg_bf16_t128_bf16(const lcma::PlaneGemmParams *p, void *stream);
static lcma::PlaneGemmParams wide_tiles(const lcma::FewRowsParams &p) {
    lcma::PlaneGemmParams q{};
    q.A = p.A;
    q.B = p.W;
    q.C = p.C;
    q.a_bytes = p.a_bytes;
    q.b_bytes = p.w_bytes;
    q.c_bytes = p.c_bytes;
    q.lda_b = p.lda_b;
    q.ldb_b = p.ldw_b;
    q.ldc_b = p.ldc_b;
    q.n_row_b = p.n_row_b;
    q.ny = p.steps / 2;
    q.tail_b = 128;
    q.nx = p.row_blocks;
    q.nz = p.partial_ld / 128;
    q.panel = p.panel;
    q.jobs = q.nx * q.nz;
    q.interleave = 5;
    return q;
}
#define LCMA_FEW_ROWS_TYPE(NAME, KIND)                                                                                 \
    LCMA_FEW_ROWS_KERNEL(NAME##_16, KIND, 16, 4, 2)                                                                    \
    LCMA_FEW_ROWS_KERNEL(NAME##_16_deep, KIND, 16, 8, 4)                                                               \
    extern "C" int lcma_launch_few_rows_##NAME##_16(const lcma::FewRowsParams *p, int grid, void *stream) {            \
        if (p->deep) lcma_k_few_rows_##NAME##_16_deep<<<dim3(grid), dim3(512), 0, (hipStream_t)stream>>>(*p);          \
        else lcma_k_few_rows_##NAME##_16<<<dim3(grid), dim3(256), 0, (hipStream_t)stream>>>(*p);                       \
        return (int)hipGetLastError();                                                                                 \
    }                                                                                                                  \
    LCMA_FEW_ROWS(NAME##_32, KIND, 32, 4, 2)                                                                           \
    LCMA_FEW_ROWS_KERNEL(NAME##_64, KIND, 64, 4, 2)                                                                    \
    extern "C" int lcma_launch_few_rows_##NAME##_64(const lcma::FewRowsParams *p, int grid, void *stream) {            \
        if (p->deep) {                                                                                                 \
            const lcma::PlaneGemmParams q = wide_tiles(*p);                                                            \
            return lcma_launch_pg_##NAME##_t128_##NAME(&q, stream);                                                    \
        }                                                                                                              \
        lcma_k_few_rows_##NAME##_64<<<dim3(grid), dim3(256), 0, (hipStream_t)stream>>>(*p);                            \
        return (int)hipGetLastError();                                                                                 \
    }                                                                                                                  \
    extern "C" __global__ __launch_bounds__(256) void lcma_k_few_rows_sum_##NAME(const lcma::FewRowsParams p) {        \
        few_rows_sum<KIND>(p);                                                                                         \
    }                                                                                                                  \
    extern "C" int lcma_launch_few_rows_sum_##NAME(const lcma::FewRowsParams *p, int rows, void *stream) {             \
        lcma_k_few_rows_sum_##NAME<<<dim3((p->n_row_b / 8 + 255) / 256, rows), dim3(256), 0, (hipStream_t)stream>>>(*p); \
        return (int)hipGetLastError();                                                                                 \
    }

LCMA_FEW_ROWS_TYPE(f16, F16)
LCMA_FEW_ROWS_TYPE(bf16, BF16)
