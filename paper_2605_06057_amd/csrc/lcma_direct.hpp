// Fused LCMA kernel for small fp32 products on gfx950: fragments from memory straight into registers, K split between waves.
//
// The staged kernels (lcma_device.hpp) give a group to a work-group of four waves that walk all of K/k together: 256^3 with
// <2,2,2;7> is four work-groups on 256 CUs, each bound by its own matrix pipes.  Here a group is a tile of 16 MI x 16 NI of
// every block and the KS waves of its work-group split K/k between them, 16 elements at a time.  Waves share nothing, so
// nothing is staged and no barrier stands in the loop: a lane reads 16 bytes of a row of A_{i,l} (and of W), or the NI
// neighbouring columns of a row of B_{l,j}, and the combinations of Eq. 3 / Eq. 4 are formed on the fragments as in the
// fragment-combine kernels.  Behind the loop every wave applies W (Eq. 6) to its own sums (it is linear), the KS partial tiles
// of the blocks of C are added in LDS in ascending wave order and stored as 16-byte vectors.
// What bounds it: the matrix pipe (16x16x4, 32 cycles; 28 MI NI of them per 16 elements of K against at most 20 MI + 8 NI
// loads), behind a start of about 4 us.  Which k meets which lane is the same for both layouts of B, so both give the same bits.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lcma_prepare_b.hpp" // for_each_const

namespace lcma {

// CH (generated): the blocks, products and combinations of the scheme, as in run_chunk; CHH (generated): NC outputs with c_i, c_j
// and the sum over the products.  TB: B is the N x K matrix W; PB: the planes of the offline Combine B (one fragment per product,
// nothing to combine: the sums of Eq. 4 were rounded to fp32 there as they are here).
template <int MI, int NI, int KS, bool TB, bool PB, class CH, class CHH> struct Direct {
    static constexpr bool ROWS_B = TB || PB; // the rows of B are k-contiguous; a fragment is 16 of them
    static constexpr int TM = 16 * MI, TN = 16 * NI, NC = CHH::NC;
    static constexpr int PITCH = TN + 4; // floats
    static constexpr int LDS_BYTES = KS * NC * TM * PITCH * 4;
    static_assert(LDS_BYTES <= 160 * 1024, "LDS budget of one CU");

    static LCMA_DEV void run(const Params &p, LCMA_LDS char *lds) {
        const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int x = blockIdx.x / p.nz, z = blockIdx.x % p.nz;
        const auto ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.A), 0, (int)p.a_bytes, 0x00020000);
        const auto rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.B), 0, (int)p.b_bytes, 0x00020000);
        const auto rc = __builtin_amdgcn_make_buffer_rsrc(p.C, 0, (int)p.c_bytes, 0x00020000);
        // rows past M (and, as W, past N) and rows of B past K lie past the extents and read as zero; columns that would alias the
        // next row are sent there: columns of B past N here, columns of A (and W) past K in the loop
        uint32_t a_row[MI], b_row[NI], b_col[CH::NB ? CH::NB : 1];
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) a_row[mi] = (uint32_t)(x * TM + mi * 16 + r) * p.lda_b + q * 16;
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) b_row[ni] = (uint32_t)(z * TN + ni * 16 + r) * p.ldb_b + q * 16; // (ROWS_B)
        if constexpr (!ROWS_B) {
#pragma unroll
            for (int t = 0; t < CH::NB; ++t) { // (K x N: column z TN + NI r + ni)
                const uint32_t colb = (uint32_t)CH::b_j(t) * p.b_bcol + (uint32_t)(z * TN + NI * r) * 4;
                b_col[t] = colb < p.n_row_b ? colb + (uint32_t)(q * 4) * p.ldb_b : p.b_bytes;
            }
        }
        f32x4 h[CH::NP][MI][NI];
        for_each_const<CH::NP>([&](auto s) {
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) h[s][mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};
        });
        for (int y = w; y < p.ny; y += KS) {
            f32x4 a[MI][CH::NA], b[NI][CH::NB ? CH::NB : 1];
            const uint32_t yb = (uint32_t)y * 64; // byte column of the 16 elements in a block of A (or W)
#pragma unroll
            for (int t = 0; t < CH::NA; ++t) {
                const uint32_t off = (uint32_t)CH::a_l(t) * p.a_bcol + yb;
                const bool in = off + q * 16 < p.k_row_b;
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
                    a[mi][t] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                             ra, (int)(in ? a_row[mi] : p.a_bytes), (int)((uint32_t)CH::a_i(t) * p.a_brow + off), 0));
            }
            if constexpr (!PB) {
#pragma unroll
                for (int t = 0; t < CH::NB; ++t) {
                    if constexpr (TB) {
                        const uint32_t off = (uint32_t)CH::b_l(t) * p.b_brow + yb; // (b_brow: byte step along K of W)
                        const bool in = off + q * 16 < p.k_row_b;
#pragma unroll
                        for (int ni = 0; ni < NI; ++ni)
                            b[ni][t] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                                     rb, (int)(in ? b_row[ni] : p.b_bytes), (int)((uint32_t)CH::b_j(t) * p.b_bcol + off), 0));
                    } else {
                        const uint32_t off = (uint32_t)CH::b_l(t) * p.b_brow + (uint32_t)y * 16 * p.ldb_b;
#pragma unroll
                        for (int e = 0; e < 4; ++e) { // row 16 y + 4 q + e
                            const uint32_t at = off + (uint32_t)e * p.ldb_b;
                            if constexpr (NI == 1) {
                                const uint32_t v = __builtin_amdgcn_raw_buffer_load_b32(rb, (int)b_col[t], (int)at, 0);
                                b[0][t][e] = __builtin_bit_cast(float, v);
                            } else {
                                static_assert(NI == 2, "one or two columns per lane");
                                typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                                const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rb, (int)b_col[t], (int)at, 0);
                                const uint32_t v0 = v[0], v1 = v[1];
                                b[0][t][e] = __builtin_bit_cast(float, v0);
                                b[1][t][e] = __builtin_bit_cast(float, v1);
                            }
                        }
                    }
                }
            }
            f32x4 ca[MI][CH::NP], cb[NI][CH::NP];
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) CH::comb_a(a[mi], ca[mi]);
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                if constexpr (PB) { // (the planes are padded with zeros: no column is past K)
#pragma unroll
                    for (int s = 0; s < CH::NP; ++s)
                        cb[ni][s] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                                  rb, (int)b_row[ni], (int)((uint32_t)CH::b_plane(s) * p.b_brow + yb), 0));
                } else {
                    CH::comb_b(b[ni], cb[ni]);
                }
            }
            for_each_const<CH::NP>([&](auto s) {
#pragma unroll
                for (int e = 0; e < 4; ++e) // (element e of lane group q: k = 4 q + e)
#pragma unroll
                    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                        for (int ni = 0; ni < NI; ++ni)
                            h[s][mi][ni] = __builtin_amdgcn_mfma_f32_16x16x4f32(ca[mi][s][e], cb[ni][s][e], h[s][mi][ni], 0, 0, 0);
            });
        }
        // partial blocks of C: accumulator value v is row 4 q + v, column r of its 16 x 16 tile
        LCMA_LDS float *mine = (LCMA_LDS float *)lds + w * (NC * TM * PITCH);
        for_each_const<NC>([&](auto o) {
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) {
                    const f32x4 c = CHH::comb(h, o, mi, ni);
#pragma unroll
                    for (int v = 0; v < 4; ++v) mine[(o * TM + mi * 16 + 4 * q + v) * PITCH + (ROWS_B ? ni * 16 + r : NI * r + ni)] = c[v];
                }
        });
        __syncthreads();
        for (int t = threadIdx.x; t < NC * TM * TN / 4; t += 64 * KS) {
            const int col = t % (TN / 4) * 4, row = t / (TN / 4) % TM, o = t / (TN / 4 * TM);
            const LCMA_LDS float *at = (const LCMA_LDS float *)lds + (o * TM + row) * PITCH + col;
            f32x4 sum = *(const LCMA_LDS f32x4 *)at;
#pragma unroll
            for (int k = 1; k < KS; ++k) sum += *(const LCMA_LDS f32x4 *)(at + k * (NC * TM * PITCH));
            const uint32_t colb = (uint32_t)CHH::c_j(o) * p.c_bcol + (uint32_t)(z * TN + col) * 4;
            // vectors past N go to the end of the extent and are dropped, rows past M lie past it
            const uint32_t off = colb < p.n_row_b ? (uint32_t)CHH::c_i(o) * p.c_brow + (uint32_t)(x * TM + row) * p.ldc_b + colb : p.c_bytes;
            sum *= p.alpha;
            if (p.beta != 0.f) {
                const f32x4 old = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rc, (int)off, 0, 0));
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[e] = __builtin_fmaf(p.beta, old[e], sum[e]);
            }
            // (16-byte store: the scalar-offset field stays a literal zero, see Ctx::store_c in lcma_device.hpp)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, sum), rc, (int)off, 0, 0);
        }
    }
};

} // namespace lcma
