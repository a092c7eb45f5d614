// Plain C = A x W^T for few rows of A or a small C (16-bit storage, N x K weights), for gfx950.
//
// With M of a few dozen the product is bound by reading W once (N K 2 bytes), not by the matrix pipe, and tiles of 128 x 128
// leave most of the chip idle: 64 x 4096 x 4096 is 32 of them, each walking all of K in 64 dependent steps.  Here a
// work-group owns a tile of 64 x 64 (32 x 32, 16 x 16) of C and its waves split K between them, a line (64 k, 128 bytes of
// every row) to a wave in turn.  Nothing is shared between waves, so there is no barrier in the loop: each wave has stages of its own in
// LDS, sends the loads of its next lines straight into them, waits for a line by count and reads its fragments.  At the end the
// partial tiles are added in LDS in ascending wave order, in fp32, and rounded once.
// What bounds it is what ONE CU can take in.  A load whose neighbouring lanes ask for one row after the other, as the fragments of the matrix
// instructions want them, takes a CU 64 clocks (38 bytes/ns, measured, 16 rows x 64 bytes and 32 x 32 alike); with eight lanes to the
// 128 bytes of a row it takes 16 (140 to 150 from the L2, 100 with all CUs at it).  So lines travel whole into LDS and the fragments are read there.
// The bytes per work-group decide next: a large tile of C reads least in all, and when large tiles alone would not fill the chip
// K is cut into slices for work-groups of their own, whose fp32 partial products a second kernel adds in ascending order
// (four slices of 64 x 4096: 4.5 us).
// What a work-group holds in LDS decides how many of them a CU runs: four waves with two lines in flight each, 32, 64 and 128 KB for tiles of 16,
// 32 and 64, so that the many work-groups of the smaller tiles run side by side (16 x 8192 x 512, 512 of them: 3.9 us, 6.0 with 128 KB;
// 1 x 14336 x 1024, 896: 7.6 / 12.1; tiles of 32 with 128 KB, eight waves: 256 x 1024 x 1024 5.0, now 4.4).
// Measured (bf16, us, fragments from memory straight into registers / this): 64 x 4096 x 4096 in four slices 14.9 / 13.3, in one piece
// 17.3 / 9.0 (tiles of 32, what the rule takes); 64 x 4096 x 14336 37 / 30 (117 MB of weights: 3.9 TB/s); 64 x 14336 x 4096 37 / 28; 128 x 4096 x 4096 21.6 / 14.3; 1 x 14336 x
// 4096 25.5 / 23.1; 256 x 1024 x 1024 6.5 / 4.4; 65 x 4088 x 4160 23.6 / 14.3.  Few columns (fp16): 4266 x 128 x 4288 33 / 16.6, 4095 x 192 x 2176 19.3 / 11.2
// (97 and 37 with the blocks of columns dealt to the XCDs one by one, which leaves most XCDs without work where there are fewer than eight).
// Where there would be two tiles of 64 x 64 to a CU, 64 x 128 on csrc/lcma_kpair.hpp: 512 x 4096 x 4096 29.5 / 22.3, 320 x 4096 x 4096 28 / 19.3.
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

template <> struct Mma16<F32> { // (no tiles of 16 in fp32: the fragment alone)
    using frag = f32x4;
};

// s_waitcnt for all but the N youngest vector memory instructions; nothing moves across it
template <int N> LCMA_DEV void wait_loads() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt((N & 15) | (N >> 4) << 14 | 0x0F70);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// T: rows and columns of the tile of C; WK waves, all along K; S lines of 128 bytes of every row (64 k, fp32: 32) of a wave in flight.
// KN: the right operand is B, K x N: a line of it is its rows (k) of T columns, and the fragments of 16-bit types are read with the transposing
// LDS read.  TAIL: K may end inside a line.  Either layout adds the same terms in the same order.
template <class KIND, int T, int WK, int S, bool KN = false, bool TAIL = KN> struct FewRows {
    static constexpr int F = T == 16 ? 16 : 32, NF = T / F, KF = 64 / (512 / F); // 16x16x32 or 32x32x16 instructions; fragments of a line along K
    static constexpr int ES = KIND::ES, LINE_K = 128 / ES;
    static_assert(T >= 32 || (!KN && ES == 2), "tiles of 16: rows of 16-bit weights");
    static constexpr int LOADS = T / 8, HALF = T * 128, STAGE = 2 * HALF;         // direct loads of 1 KB and bytes of a line of either operand
    static constexpr int PITCH = T + 4;                                           // (floats; 4: the row groups of a write meet different banks)
    static constexpr int SUMS = WK * T * PITCH * 4, STAGES = WK * S * STAGE, LDS_BYTES = SUMS > STAGES ? SUMS : STAGES;
    static_assert(LDS_BYTES <= 160 * 1024 && (S == 2 || S == 4) && 2 * LOADS * S <= 63, "LDS budget of one CU; counter of loads");
    using Frag = typename Mma16<KIND>::frag;
    using Acc = std::conditional_t<F == 16, f32x4, f32x16>;

    static LCMA_DEV void run(const FewRowsParams &p, LCMA_LDS char *lds) {
        const int lane = threadIdx.x & 63, fr = lane & (F - 1), fk = lane / F;
        const int wk = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        // an eighth of the work-groups to every XCD (they go to the eight in turn), cut along the longer side of C and, first, along K: an
        // XCD reads its part of the longer operand alone and few slices of the other one
        const int col_blocks = p.partial_ld / T, jobs = col_blocks * p.slices, groups = jobs * p.row_blocks; // (groups: the grid)
        const int share = (groups + 7) / 8, left = groups % 8, xcd = blockIdx.x % 8;
        const int id = (left && xcd > left ? left * share + (xcd - left) * (share - 1) : xcd * share) + blockIdx.x / 8;
        const bool tall = p.row_blocks * T > p.partial_ld;
        const int inner = tall ? jobs : p.row_blocks, hi = id / inner, lo = id - hi * inner;
        const int mb = tall ? hi : lo, job = tall ? lo : hi, slice = job / col_blocks, cb = job - slice * col_blocks;
        const int lines = p.steps / 2, per = p.slice_steps / 2, first = slice * per, end = first + per < lines ? first + per : lines;
        Acc acc[NF][NF];
#pragma unroll
        for (int i = 0; i < NF; ++i)
#pragma unroll
            for (int j = 0; j < NF; ++j)
#pragma unroll
                for (int v = 0; v < F * F / 64; ++v) acc[i][j][v] = 0.f;
        LCMA_LDS char *st = lds + wk * (S * STAGE);
        lines_of_wave(p, mb, cb, first + wk, end, acc, st, st + STAGE, st + (S == 4 ? 2 * STAGE : 0), st + (S == 4 ? 3 * STAGE : 0));
        __syncthreads(); // no load is in flight and every wave has read its last line: the partial tiles take the place of the stages
        LCMA_LDS float *mine = (LCMA_LDS float *)lds + wk * (T * PITCH);
#pragma unroll
        for (int i = 0; i < NF; ++i)
#pragma unroll
            for (int j = 0; j < NF; ++j)
#pragma unroll
                for (int v = 0; v < F * F / 64; ++v) mine[(i * F + (v >> 2) * 8 + fk * 4 + (v & 3)) * PITCH + j * F + fr] = acc[i][j][v];
        __syncthreads();
        const auto rc = __builtin_amdgcn_make_buffer_rsrc(p.C, 0, (int)p.c_bytes, 0x00020000);
        for (int t = threadIdx.x; t < T * T / 4; t += 64 * WK) { // four neighbouring columns
            const int row = t / (T / 4), col = t % (T / 4) * 4;
            const LCMA_LDS float *at = (const LCMA_LDS float *)lds + row * PITCH + col;
            f32x4 sum = *(const LCMA_LDS f32x4 *)at;
#pragma unroll
            for (int k = 1; k < WK; ++k) sum += *(const LCMA_LDS f32x4 *)(at + k * T * PITCH);
            const int m = mb * T + row;
            if (p.slices > 1) { // (the second kernel adds the slices)
                *(f32x4 *)((float *)p.partial + ((int64_t)slice * p.row_blocks * T + m) * p.partial_ld + cb * T + col) = sum;
            } else {
                const uint32_t colb = (uint32_t)(cb * T + col) * ES;
                const uint32_t off = colb < p.n_row_b ? (uint32_t)m * p.ldc_b + colb : p.c_bytes; // rows past M: past the extent
                if constexpr (ES == 4) {
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, sum), rc, (int)off, 0, 0);
                } else {
                    const u32x2 v = {Round<KIND>::run(sum[0]) | (Round<KIND>::run(sum[1]) << 16), Round<KIND>::run(sum[2]) | (Round<KIND>::run(sum[3]) << 16)};
                    __builtin_amdgcn_raw_buffer_store_b64(v, rc, (int)off, 0, 0);
                }
            }
        }
    }
    // KN, 16-bit: chunk c of row k of a line sits at position c ^ column_swizzle(k), so that the four rows of a transposing read meet different
    // banks (rows of 64 bytes do so by themselves).
    static LCMA_DEV constexpr int column_swizzle(int k) { return KN && ES == 2 && T == 64 ? (k >> 1 & 1) * 4 : 0; }
    // Fragments of 32 columns, 32 block and on, of a line (64 rows of T columns); as read_columns of lcma_pingpong.hpp, whose rows are 256 bytes.
    static LCMA_DEV void read_columns(const LCMA_LDS char *line, int block, Frag (&f)[KF]) {
        constexpr int P = T * 2;
        const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4, k = i >> 2, c = block * 4 + (g & 1) * 2 + ((i & 3) >> 1);
        const uint32_t at = (uint32_t)(uintptr_t)line + ((g >> 1) * 8 + k) * P + (c ^ column_swizzle(k)) * 16 + (i & 1) * 8;
        u32x2 r[4][2];
        asm volatile("ds_read_b64_tr_b16 %0, %8\n"
                     "ds_read_b64_tr_b16 %1, %8 offset:%9\n"
                     "ds_read_b64_tr_b16 %2, %8 offset:%10\n"
                     "ds_read_b64_tr_b16 %3, %8 offset:%11\n"
                     "ds_read_b64_tr_b16 %4, %8 offset:%12\n"
                     "ds_read_b64_tr_b16 %5, %8 offset:%13\n"
                     "ds_read_b64_tr_b16 %6, %8 offset:%14\n"
                     "ds_read_b64_tr_b16 %7, %8 offset:%15\n"
                     "s_waitcnt lgkmcnt(0)"
                     : "=&v"(r[0][0]), "=&v"(r[0][1]), "=&v"(r[1][0]), "=&v"(r[1][1]), "=&v"(r[2][0]), "=&v"(r[2][1]), "=&v"(r[3][0]), "=&v"(r[3][1])
                     : "v"(at), "n"(4 * P), "n"(16 * P), "n"(20 * P), "n"(32 * P), "n"(36 * P), "n"(48 * P), "n"(52 * P)
                     : "memory");
#pragma unroll
        for (int j = 0; j < 4; ++j) f[j] = __builtin_bit_cast(Frag, u32x4{r[j][0][0], r[j][0][1], r[j][1][0], r[j][1][1]});
    }
    // Lines `line`, line + WK, ... below `end` of tile (mb, cb).  s0 .. s3: the stages of the wave.  restrict: the loads in flight towards
    // one do not touch what is read from another (the compiler would otherwise wait for all of them in front of every read).  It holds
    // in here only: the partial tiles, which take the place of the stages, are written where it has ended.
    static LCMA_DEV void lines_of_wave(const FewRowsParams &p, int mb, int cb, int line, int end, Acc (&acc)[NF][NF], LCMA_LDS char *__restrict__ s0,
                                       LCMA_LDS char *__restrict__ s1, LCMA_LDS char *__restrict__ s2, LCMA_LDS char *__restrict__ s3) {
        const int lane = threadIdx.x & 63, fr = lane & (F - 1), fk = lane / F;
        const auto ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.A), 0, (int)p.a_bytes, 0x00020000);
        const auto rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.W), 0, (int)p.w_bytes, 0x00020000);
        // A load brings 8 rows of 128 bytes, lanes 8 i to 8 i + 7 one row.  Rows past M or N lie past the extents and read as zero; 16-byte
        // chunk c of row i sits at position c ^ (i / 2 % 8), so that 16 rows at one chunk column meet all banks once.
        uint32_t av[2], bv[2], at[2], bt[2]; // even and odd loads of a line (at, bt: of the last one, what is past K from past the extents)
        const int lines = p.steps / 2;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t c = ((lane & 7) ^ (lane >> 4) ^ (4 * i)) * 16;
            av[i] = (uint32_t)(mb * T + (lane >> 3)) * p.lda_b + c;
            bv[i] = (uint32_t)(cb * T + (lane >> 3)) * p.ldw_b + c;
            at[i] = TAIL && c >= p.tail_b ? p.a_bytes : av[i];
            bt[i] = TAIL && c >= p.tail_b ? p.w_bytes : bv[i];
        }
        constexpr int CPR = T * ES / 16, RPL = 64 / CPR; // KN: 16-byte chunks of a row (k) of the line, rows of a load
        if constexpr (KN) bv[0] = (uint32_t)(lane / CPR) * p.ldw_b + (uint32_t)(cb * T) * ES + ((lane % CPR) ^ column_swizzle(lane / CPR)) * 16; // (rows past K: past the extent)
        auto load = [&](LCMA_LDS char *st, int line) { // a line past the end is read from the end of the extents: zeros
            const bool in = line < end, last = TAIL && line + 1 == lines;
            const uint32_t ka = in ? (uint32_t)line * 128 : p.a_bytes, kb = in ? (uint32_t)line * (KN ? LINE_K * p.ldw_b : 128) : p.w_bytes;
#pragma unroll
            for (int i = 0; i < LOADS; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (LCMA_LDS void *)(st + i * 1024), 16, (int)(last ? at[i & 1] : av[i & 1]), (int)(ka + i * 8 * p.lda_b), 0, 0);
#pragma unroll
            for (int i = 0; i < LOADS; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (LCMA_LDS void *)(st + HALF + i * 1024), 16, (int)(KN ? bv[0] : last ? bt[i & 1] : bv[i & 1]), (int)(kb + i * (KN ? RPL : 8) * p.ldw_b), 0, 0);
        };
        uint32_t frag[KF]; // of this lane's 16 bytes in either operand's rows
#pragma unroll
        for (int k = 0; k < KF; ++k) frag[k] = fr * 128 + ((k * (64 / F) + fk) ^ (fr >> 1 & 7)) * 16;
        auto step = [&](LCMA_LDS char *st, int line) {
            Frag a[KF][NF], b[KF][NF];
            wait_loads<2 * LOADS *(S - 1)>();
#pragma unroll
            for (int k = 0; k < KF; ++k)
#pragma unroll
                for (int i = 0; i < NF; ++i) {
                    a[k][i] = __builtin_bit_cast(Frag, *(const LCMA_LDS u32x4 *)(st + frag[k] + i * F * 128));
                    if constexpr (!KN) b[k][i] = __builtin_bit_cast(Frag, *(const LCMA_LDS u32x4 *)(st + HALF + frag[k] + i * F * 128));
                    else if constexpr (ES == 4)
#pragma unroll
                        for (int t = 0; t < 4; ++t) b[k][i][t] = *(const LCMA_LDS float *)(st + HALF + ((k * 2 + fk) * 4 + t) * (T * ES) + (i * F + fr) * 4);
                }
            if constexpr (KN && ES == 2)
#pragma unroll
                for (int i = 0; i < NF; ++i) {
                    Frag col[KF];
                    read_columns(st + HALF, i, col);
#pragma unroll
                    for (int k = 0; k < KF; ++k) b[k][i] = col[k];
                }
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(0xC07F); // lgkmcnt(0): what was read has left LDS, so its place may be loaded anew
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
            load(st, line + S * WK);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < KF; ++k)
#pragma unroll
                for (int i = 0; i < NF; ++i)
#pragma unroll
                    for (int j = 0; j < NF; ++j) {
                        if constexpr (F == 16) acc[i][j] = Mma16<KIND>::run(a[k][i], b[k][j], acc[i][j]);
                        else Mma<KIND>::run(a[k][i], b[k][j], acc[i][j]);
                    }
        };
        load(s0, line);
        load(s1, line + WK);
        if constexpr (S == 4) {
            load(s2, line + 2 * WK);
            load(s3, line + 3 * WK);
        }
        while (line < end) {
            step(s0, line);
            if ((line += WK) >= end) break;
            step(s1, line);
            if constexpr (S == 4) {
                if ((line += WK) >= end) break;
                step(s2, line);
                if ((line += WK) >= end) break;
                step(s3, line);
            }
            line += WK;
        }
        wait_loads<0>();
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
