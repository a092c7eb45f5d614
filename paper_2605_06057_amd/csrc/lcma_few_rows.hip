// Instances of the plain product on few rows (csrc/lcma_few_rows.hpp) and of the kernel that adds the slices of K.
#include "lcma_few_rows.hpp"

using namespace lcma;

#define LCMA_FEW_ROWS(NAME, KIND, T, WK, S)                                                                             \
    extern "C" __global__ __launch_bounds__(64 * WK, 1) void lcma_k_few_rows_##NAME(const lcma::FewRowsParams p) {         \
        using G = FewRows<KIND, T, WK, S>;                                                                            \
        __shared__ __attribute__((aligned(16))) char smem[G::LDS_BYTES];                                               \
        G::run(p, (LCMA_LDS char *)smem);                                                                              \
    }                                                                                                                  \
    extern "C" int lcma_launch_few_rows_##NAME(const lcma::FewRowsParams *p, int grid, void *stream) {                 \
        lcma_k_few_rows_##NAME<<<dim3(grid), dim3(64 * WK), 0, (hipStream_t)stream>>>(*p);                                 \
        return (int)hipGetLastError();                                                                                 \
    }
#define LCMA_FEW_ROWS_TYPE(NAME, KIND)                                                                                 \
    LCMA_FEW_ROWS(NAME##_16, KIND, 16, 8, 4)                                                                            \
    LCMA_FEW_ROWS(NAME##_32, KIND, 32, 8, 2)                                                                            \
    LCMA_FEW_ROWS(NAME##_64, KIND, 64, 4, 2)                                                                            \
    extern "C" __global__ __launch_bounds__(256) void lcma_k_few_rows_sum_##NAME(const lcma::FewRowsParams p) {        \
        few_rows_sum<KIND>(p);                                                                                         \
    }                                                                                                                  \
    extern "C" int lcma_launch_few_rows_sum_##NAME(const lcma::FewRowsParams *p, int rows, void *stream) {             \
        lcma_k_few_rows_sum_##NAME<<<dim3((p->n_row_b / 8 + 255) / 256, rows), dim3(256), 0, (hipStream_t)stream>>>(*p); \
        return (int)hipGetLastError();                                                                                 \
    }

LCMA_FEW_ROWS_TYPE(f16, F16)
LCMA_FEW_ROWS_TYPE(bf16, BF16)
