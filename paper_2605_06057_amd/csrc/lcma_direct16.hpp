// Fused LCMA kernel for 16-bit products with few tiles on gfx950: the sibling of lcma_direct.hpp for fp16 and bf16 storage.
//
// The staged kernels give a group of 64 x 64 blocks to one work-group that walks all of K/k in dependent steps of 32: 1000 x 1544 x
// 2056 with <2,2,2;7> is 104 work-groups of 33 steps at 1 us, 239 x 2176 x 9024 is 36 of 141.  Here a group is a tile of 16 x 64 of
// every block and the KS waves of its work-group split K/k between them, a step of 64 to a wave in turn.  Waves share nothing:
// fragments come from memory straight into registers, one step ahead of the matrix instructions, are converted and combined there
// (the same conversions and sums as the fragment-combine kernels), and the partial tiles of C are added in LDS in ascending wave
// order, in fp32, and rounded once.
// Tile and step: a lane's 16 elements of a row are the two halves of one 32-byte piece, so that both fragments of a step take whole
// 128-byte lines of A (and of W); 64 columns are a whole line of B.  Which k meets which lane is the same for both layouts of
// B, so both give the same bits.
// What bounds it: a load instruction takes a CU about 26 clocks wherever the line comes from (48 bytes/ns), 2.6 to 4.2 us for a step of
// four waves, N x K 2.9 to 4.6 (16 bytes per lane of 16 rows: see SWAP).  Measured (us, staged 64 x 64 x 32 against this; three sets
// of operands in turn, launches from a graph), K x N bf16, N x K bf16, N x K fp16: 239 x 2176 x 9024 133 / 63, 108 / 75, 85 / 66;
// 473 x 344 x 2696 45 / 27, 41 / 28, 41 / 25; 64 x 4096 x 4096 65 / 33, 53 / 36, 41 / 33; 1024^3 21.1 / 15.4, 18.2 / 15.1, 15.9 /
// 15.6.  With more than a round of 256 work-groups the larger tiles win: 1000 x 1544 x 2056 37 / 44, 33 / 46, 33 / 41.  Two or four
// waves side by side along M, one step apart in time, so that they ask for the same lines of B together: 156 and 304 at 239 x 2176
// x 9024 (fewer waves along K, no line saved).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lcma_prepare_b.hpp" // for_each_const

namespace lcma {

// IN: storage type.  CH, CHH (generated): as for Direct.  TB: B is the N x K matrix W.
template <class IN, int KS, bool TB, class CH, class CHH> struct Direct16 {
    static constexpr int NI = 4, TM = 16, TN = 16 * NI, NC = CHH::NC;
    static constexpr int PITCH = TN + 4; // floats
    static constexpr int LDS_BYTES = KS * NC * TM * PITCH * 4;
    static_assert(LDS_BYTES <= 160 * 1024, "LDS budget of one CU");
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

    struct Batch { // one step: two fragments of every block of A and of every 16 columns of a block of B
        u32x4 a[2][CH::NA], b[2][CH::NB][TB ? NI : 1];
        u32x2 c[2][CH::NB][TB ? 1 : 8]; // (K x N: four columns of eight rows)
    };

    static LCMA_DEV void run(const Params &p, LCMA_LDS char *lds) {
        if (TB && p.ldb_b % 128 == 0) body<true>(p, lds);
        else body<false>(p, lds);
    }

    // SWAP (rows of W that all start at the same place of a line): neighbouring lanes would ask for the same 16 bytes of two lines,
    // which the L1 cache serves one after the other.  So the odd rows read the second half of their 32 bytes first, and the
    // halves change places in registers (fp16, without / with: 101 x 456 x 1024 16.5 / 12.5 us, 57 x 3488 x 7168 69 / 54; rows
    // that start anywhere else 25 / 26, where the exchange would only cost).
    template <bool SWAP> static LCMA_DEV void body(const Params &p, LCMA_LDS char *lds) {
        const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        // an eighth of the tiles to every XCD (work-groups go to the eight in turn), cut along the longer side of C, so that the
        // longer operand is read by one XCD only
        const int share = (gridDim.x + 7) / 8, left = gridDim.x % 8, xcd = blockIdx.x % 8;
        const int id = (left && xcd > left ? left * share + (xcd - left) * (share - 1) : xcd * share) + blockIdx.x / 8;
        const bool wide = p.nz * TN >= p.nx * TM;
        const int x = wide ? id % p.nx : id / p.nz, z = wide ? id / p.nx : id % p.nz;
        const auto ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.A), 0, (int)p.a_bytes, 0x00020000);
        const auto rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.B), 0, (int)p.b_bytes, 0x00020000);
        const auto rc = __builtin_amdgcn_make_buffer_rsrc(p.C, 0, (int)p.c_bytes, 0x00020000);
        // rows past M (and, as W, past N) and rows of B past K lie past the extents and read as zero; columns that would alias the
        // next row are sent there: columns of B past N here, columns of A (and W) past K with every load
        const uint32_t a_row = (uint32_t)(x * TM + r) * p.lda_b + q * 32;
        uint32_t b_row[NI], b_col[CH::NB];
        if constexpr (TB) {
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) b_row[ni] = (uint32_t)(z * TN + ni * 16 + r) * p.ldb_b + q * 32;
        } else {
#pragma unroll
            for (int t = 0; t < CH::NB; ++t) { // column z TN + 4 r + ni
                const uint32_t colb = (uint32_t)CH::b_j(t) * p.b_bcol + (uint32_t)(z * TN + NI * r) * 2;
                b_col[t] = colb < p.n_row_b ? colb + (uint32_t)(q * 16) * p.ldb_b : p.b_bytes;
            }
        }
        auto load = [&](Batch &m, int y) {
#pragma unroll
            for (int t = 0; t < CH::NA; ++t) {
                const uint32_t off = (uint32_t)CH::a_l(t) * p.a_bcol + (uint32_t)y * 128;
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    m.a[u][t] = __builtin_amdgcn_raw_buffer_load_b128(ra, (int)(off + q * 32 + u * 16 < p.k_row_b ? a_row : p.a_bytes),
                                                                      (int)((uint32_t)CH::a_i(t) * p.a_brow + off + u * 16), 0);
            }
#pragma unroll
            for (int t = 0; t < CH::NB; ++t) {
                if constexpr (TB) {
                    const uint32_t off = (uint32_t)CH::b_l(t) * p.b_brow + (uint32_t)y * 128; // (b_brow: byte step along K of W)
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            const uint32_t at = off + (SWAP ? 0 : u * 16), half = !SWAP ? 0 : r & 1 ? 16 - u * 16 : u * 16;
                            m.b[u][t][ni] = __builtin_amdgcn_raw_buffer_load_b128(rb, (int)(at + q * 32 + half < p.k_row_b ? b_row[ni] + half : p.b_bytes),
                                                                                  (int)((uint32_t)CH::b_j(t) * p.b_bcol + at), 0);
                        }
                } else {
                    const uint32_t off = (uint32_t)CH::b_l(t) * p.b_brow + (uint32_t)y * 64 * p.ldb_b;
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int e = 0; e < 8; ++e) // row 64 y + 16 q + 8 u + e
                            m.c[u][t][e] = __builtin_amdgcn_raw_buffer_load_b64(rb, (int)b_col[t], (int)(off + (uint32_t)(u * 8 + e) * p.ldb_b), 0);
                }
            }
        };
        f32x4 h[CH::NP][1][NI];
        for_each_const<CH::NP>([&](auto s) {
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) h[s][0][ni] = f32x4{0.f, 0.f, 0.f, 0.f};
        });
        auto multiply = [&](const Batch &m) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                f16x8 a[CH::NA], ca[CH::NP];
#pragma unroll
                for (int t = 0; t < CH::NA; ++t) a[t] = Convert<IN, F16>::run(m.a[u][t]);
                CH::comb_a(a, ca);
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) {
                    f16x8 b[CH::NB], cb[CH::NP];
#pragma unroll
                    for (int t = 0; t < CH::NB; ++t) {
                        u32x4 raw;
                        if constexpr (TB) {
                            raw = SWAP && r & 1 ? m.b[1 - u][t][ni] : m.b[u][t][ni];
                        } else {
#pragma unroll
                            for (int e = 0; e < 4; ++e) // the low or high halves of two rows
                                raw[e] = __builtin_amdgcn_perm(m.c[u][t][2 * e + 1][ni / 2], m.c[u][t][2 * e][ni / 2], ni & 1 ? 0x07060302u : 0x05040100u);
                        }
                        b[t] = Convert<IN, F16>::run(raw);
                    }
                    CH::comb_b(b, cb);
                    for_each_const<CH::NP>([&](auto s) { h[s][0][ni] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ca[s], cb[s], h[s][0][ni], 0, 0, 0); });
                }
            }
        };
        if (w < p.ny) {
            Batch even, odd;
            load(even, w);
            // past the last step of the wave: that step again, unused (offsets selected load by load: 55 -> 92 us at 239 x 2176 x 9024)
            auto next = [&](int y) { return y + KS < p.ny ? y + KS : y; };
            for (int y = w;;) {
                load(odd, next(y));
                multiply(even);
                if ((y += KS) >= p.ny) break;
                load(even, next(y));
                multiply(odd);
                if ((y += KS) >= p.ny) break;
            }
        }
        // partial blocks of C: accumulator value v is row 4 q + v, column r of its 16 x 16 tile
        LCMA_LDS float *mine = (LCMA_LDS float *)lds + w * (NC * TM * PITCH);
        for_each_const<NC>([&](auto o) {
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                const f32x4 c = CHH::comb(h, o, 0, ni);
#pragma unroll
                for (int v = 0; v < 4; ++v) mine[(o * TM + 4 * q + v) * PITCH + (TB ? ni * 16 + r : NI * r + ni)] = c[v];
            }
        });
        __syncthreads();
        for (int t = threadIdx.x; t < NC * TM * TN / 8; t += 64 * KS) {
            const int col = t % (TN / 8) * 8, row = t / (TN / 8) % TM, o = t / (TN / 8 * TM);
            const LCMA_LDS float *at = (const LCMA_LDS float *)lds + (o * TM + row) * PITCH + col;
            f32x4 sum[2] = {*(const LCMA_LDS f32x4 *)at, *(const LCMA_LDS f32x4 *)(at + 4)};
#pragma unroll
            for (int k = 1; k < KS; ++k)
#pragma unroll
                for (int i = 0; i < 2; ++i) sum[i] += *(const LCMA_LDS f32x4 *)(at + k * (NC * TM * PITCH) + 4 * i);
            const uint32_t colb = (uint32_t)CHH::c_j(o) * p.c_bcol + (uint32_t)(z * TN + col) * 2;
            // vectors past N go to the end of the extent and are dropped, rows past M lie past it
            const uint32_t off = colb < p.n_row_b ? (uint32_t)CHH::c_i(o) * p.c_brow + (uint32_t)(x * TM + row) * p.ldc_b + colb : p.c_bytes;
            sum[0] *= p.alpha;
            sum[1] *= p.alpha;
            if (p.beta != 0.f) {
                const u32x4 old = __builtin_amdgcn_raw_buffer_load_b128(rc, (int)off, 0, 0);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const uint32_t bits = old[e / 2] >> (e & 1) * 16;
                    float c;
                    if constexpr (std::is_same_v<IN, BF16>)
                        c = __builtin_bit_cast(float, bits << 16);
                    else
                        c = (float)__builtin_bit_cast(_Float16, (uint16_t)bits);
                    sum[e / 4][e % 4] = __builtin_fmaf(p.beta, c, sum[e / 4][e % 4]);
                }
            }
            u32x4 out;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                out[e] = Round<IN>::run(sum[e / 2][e % 2 * 2]) | (Round<IN>::run(sum[e / 2][e % 2 * 2 + 1]) << 16);
            // (16-byte store: the scalar-offset field stays a literal zero, see Ctx::store_c in lcma_device.hpp)
            __builtin_amdgcn_raw_buffer_store_b128(out, rc, (int)off, 0, 0);
        }
    }
};

} // namespace lcma
