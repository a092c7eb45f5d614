// Plain C = A x W^T for few rows of A or a small C (16-bit storage, N x K weights), for gfx950.
//
// With M of a few dozen the product is bound by reading W once (N K 2 bytes), not by the matrix pipe, and tiles of 128 x 128
// leave most of the chip idle: 64 x 4096 x 4096 is 32 of them, each walking all of K in 64 dependent steps.  Here a
// work-group owns a tile of 64 x 64 (32 x 32, 16 x 16) of C and its eight waves split K between them, two neighbouring steps
// of 32 elements (a 128-byte line of every row) to a wave in turn.  Nothing is shared between waves, so nothing is staged:
// fragments come from memory straight into registers, a batch of U steps ahead of the matrix instructions (16x16x32: 16 rows
// of W and 16 of A per fragment, 16 bytes per lane).  At the end the eight partial tiles are added in LDS in ascending wave
// order, in fp32, and rounded once.
// What bounds it is what ONE CU can pull in, 33 to 42 bytes/ns whatever the source (few_rows_plan takes 36): so the bytes per work-group decide, a
// large tile of C reads least in all, and when large tiles alone would not fill the chip K is cut into slices for
// work-groups of their own, whose fp32 partial products a second kernel adds in ascending order (3.7 us for its launch).
// Measured (bf16, us, against the 128 x 128 plane GEMM): 64 x 4096 x 4096 14.3 (four slices; one 31.2) against 41.4; 64 x 4096
// x 14336 36.1 against 199 (117 MB of weights: 3.3 TB/s); 64 x 14336 x 4096 35.9 (one slice) against 61.4; 128 x 4096 x 4096
// 21.5 against 42.1; 64 x 1024 x 1024 3.9 (tiles of 16) against 10.1; 256 x 1024 x 1024 5.8 (tiles of 32) against 10.1.  Few columns
// (fp16): 4266 x 128 x 4288 33 against 48, 4095 x 192 x 2176 19.6 against 24 (97 and 37 with the blocks of columns dealt to the XCDs
// one by one, which leaves most XCDs without work where there are fewer than eight).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lcma_device.hpp"

namespace lcma {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

template <class K> struct Mma16;
template <> struct Mma16<F16> {
    using frag = f16x8;
    static LCMA_DEV f32x4 run(frag a, frag b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }
};
template <> struct Mma16<BF16> {
    using frag = bf16x8;
    static LCMA_DEV f32x4 run(frag a, frag b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
};

// MT, NT: 16-row fragments of A and of W per wave; U: steps of a batch.
template <class KIND, int MT, int NT, int U> struct FewRows {
    static constexpr int WK = 8, ROWS = 16 * MT, COLS = 16 * NT; // waves, all along K; the tile of C
    static constexpr int PITCH = COLS + 4; // (floats; 4: the four row groups of a write meet different banks)
    static constexpr int LDS_BYTES = WK * ROWS * PITCH * 4;
    static_assert(LDS_BYTES <= 160 * 1024 && U % 2 == 0, "LDS budget of one CU; whole lines per batch");
    using Frag = typename Mma16<KIND>::frag;

    static LCMA_DEV void run(const FewRowsParams &p, LCMA_LDS char *lds) {
        const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
        const int wk = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const auto ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.A), 0, (int)p.a_bytes, 0x00020000);
        const auto rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.W), 0, (int)p.w_bytes, 0x00020000);
        // an eighth of the work-groups to every XCD (they go to the eight in turn), cut along the longer side of C and, first, along K: an
        // XCD reads its part of the longer operand alone and few slices of the other one
        const int col_blocks = p.partial_ld / COLS, jobs = col_blocks * p.slices, groups = jobs * p.row_blocks; // (groups: the grid)
        const int share = (groups + 7) / 8, left = groups % 8, xcd = blockIdx.x % 8;
        const int id = (left && xcd > left ? left * share + (xcd - left) * (share - 1) : xcd * share) + blockIdx.x / 8;
        const bool tall = p.row_blocks * ROWS > p.partial_ld;
        const int inner = tall ? jobs : p.row_blocks, hi = id / inner, lo = id - hi * inner;
        const int mb = tall ? hi : lo, job = tall ? lo : hi, slice = job / col_blocks, cb = job - slice * col_blocks;
        const int first = slice * p.slice_steps, end = first + p.slice_steps < p.steps ? first + p.slice_steps : p.steps;
        // rows past M or N lie past the extents and read as zero
        uint32_t a_off[MT], b_off[NT];
#pragma unroll
        for (int i = 0; i < MT; ++i) a_off[i] = (uint32_t)(mb * ROWS + i * 16 + r) * p.lda_b + q * 16;
#pragma unroll
        for (int j = 0; j < NT; ++j) b_off[j] = (uint32_t)(cb * COLS + j * 16 + r) * p.ldw_b + q * 16;
        f32x4 acc[MT][NT];
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        struct Batch {
            u32x4 a[U][MT], b[U][NT];
        };
        auto load = [&](Batch &x, int at) { // a step past the end reads from the end of the extents: zeros
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int step = at + (u >> 1) * (2 * WK) + 2 * wk + (u & 1); // (two steps are a 128-byte line of a row)
                const uint32_t ka = step < end ? (uint32_t)step * 64 : p.a_bytes, kb = step < end ? (uint32_t)step * 64 : p.w_bytes;
#pragma unroll
                for (int j = 0; j < NT; ++j) x.b[u][j] = __builtin_amdgcn_raw_buffer_load_b128(rb, (int)b_off[j], (int)kb, 0);
#pragma unroll
                for (int i = 0; i < MT; ++i) x.a[u][i] = __builtin_amdgcn_raw_buffer_load_b128(ra, (int)a_off[i], (int)ka, 0);
            }
        };
        auto multiply = [&](const Batch &x) {
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int j = 0; j < NT; ++j)
                        acc[i][j] = Mma16<KIND>::run(__builtin_bit_cast(Frag, x.a[u][i]), __builtin_bit_cast(Frag, x.b[u][j]), acc[i][j]);
        };
        Batch even, odd;
        load(even, first);
        for (int s = first;;) { // (uniform: all waves run the same number of batches)
            load(odd, s + U * WK);
            multiply(even);
            if ((s += U * WK) >= end) break;
            load(even, s + U * WK);
            multiply(odd);
            if ((s += U * WK) >= end) break;
        }
        LCMA_LDS float *mine = (LCMA_LDS float *)lds + wk * (ROWS * PITCH);
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) mine[(i * 16 + q * 4 + v) * PITCH + j * 16 + r] = acc[i][j][v];
        __syncthreads();
        const auto rc = __builtin_amdgcn_make_buffer_rsrc(p.C, 0, (int)p.c_bytes, 0x00020000);
        for (int t = threadIdx.x; t < ROWS * COLS / 4; t += 512) { // four neighbouring columns
            const int row = t / (COLS / 4), col = t % (COLS / 4) * 4;
            const LCMA_LDS float *at = (const LCMA_LDS float *)lds + row * PITCH + col;
            f32x4 sum = *(const LCMA_LDS f32x4 *)at;
#pragma unroll
            for (int k = 1; k < WK; ++k) sum += *(const LCMA_LDS f32x4 *)(at + k * ROWS * PITCH);
            const int m = mb * ROWS + row;
            if (p.slices > 1) { // (the second kernel adds the slices)
                *(f32x4 *)((float *)p.partial + ((int64_t)slice * p.row_blocks * ROWS + m) * p.partial_ld + cb * COLS + col) = sum;
            } else {
                const uint32_t colb = (uint32_t)(cb * COLS + col) * 2;
                const uint32_t off = colb < p.n_row_b ? (uint32_t)m * p.ldc_b + colb : p.c_bytes; // rows past M: past the extent
                const u32x2 v = {Round<KIND>::run(sum[0]) | (Round<KIND>::run(sum[1]) << 16), Round<KIND>::run(sum[2]) | (Round<KIND>::run(sum[3]) << 16)};
                __builtin_amdgcn_raw_buffer_store_b64(v, rc, (int)off, 0, 0);
            }
        }
    }
};

// Second kernel when K is cut into slices: adds the partial products in ascending slice order and rounds once.  A thread: four
// neighbouring columns of a row; grid.y: rows.
template <class KIND> LCMA_DEV void few_rows_sum(const FewRowsParams &p) {
    const uint32_t col = (blockIdx.x * 256 + threadIdx.x) * 4, m = blockIdx.y;
    if (col * 2 >= p.n_row_b) return;
    const float *at = (const float *)p.partial + (int64_t)m * p.partial_ld + col;
    f32x4 sum = *(const f32x4 *)at;
    for (int s = 1; s < p.slices; ++s) sum += *(const f32x4 *)(at + (int64_t)s * p.row_blocks * p.block_rows * p.partial_ld);
    const u32x2 v = {Round<KIND>::run(sum[0]) | (Round<KIND>::run(sum[1]) << 16), Round<KIND>::run(sum[2]) | (Round<KIND>::run(sum[3]) << 16)};
    *(u32x2 *)((char *)p.C + (int64_t)m * p.ldc_b + col * 2) = v;
}

} // namespace lcma
