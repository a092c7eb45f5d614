// Tiles of 128 x 128 and 64 x 128 of the plane GEMM (operands and argument block of lcma_plane_gemm.hpp), for products whose 256 x 256
// tiles would leave much of the chip idle: two groups of four waves share a tile and take the steps of 128 bytes of K in turn.
//
// What bounds a step is what a CU can take in: 32 KB of operands (24 on the lower tile) at 64 bytes a clock are 512 clocks, as long as
// the matrix instructions of the step take on the SIMDs.  PlaneGemm, in whose 128 x 128 form two work-groups of a CU read, multiply and wait as they
// come, takes 0.62 us a step.  Here
//  - the waves of a SIMD, one of each group, change roles at a barrier: while one group reads the fragments of its step (16 KB a wave: a
//    whole step of a 64 x 64 wave tile, 32 x 64 on the lower tile), the other multiplies;
//  - a group that multiplies sends the loads of its step after next in between, one to every two matrix instructions, into the stage that it
//    has just read: three slots to land, and the wait for them is a count;
//  - the two partial tiles are added at the end through LDS, each group keeping 16 of every 32 rows.
// Left out one at a time (bf16, 512 x 1024 x 8192, 32 work-groups, ns a step): as it is 302; no loads 224; no matrix instructions 297; no reads
// 300; loads only 296, and 218 where they stay in the L2.  So it waits for operands from beyond the L2; five stages instead of four (four slots to land):
// nothing.  With all 256 CUs at it 445, matrix instructions alone 273.
// Measured against the 128 x 128 tile it replaces (us): 1024 x 2048 x 4096 bf16 42.9 -> 25.2, on 64 x 128 21.6; 1352 x 1456 x 12544 133 -> 70;
// 255 x 8504 x 7296 81 -> 44; 423 x 3760 x 1344 13.9 -> 9.8; FP8 528 x 3472 x 8992 59 -> 31, 930 x 1688 x 1384 9.0 -> 6.5.  PlaneGemm stays for many tiles of few steps,
// where two work-groups to a CU hide each other's start and end.
#pragma once
#include "lcma_pingpong.hpp"

namespace lcma {

// KN (16-bit types): the right operand is B, K x N.
template <class KIND, class OUT, int TM = 128, bool KN = false> struct KPair {
    static constexpr int TN = 128, NT = 512, ROW = 128, WM = TM / 2, WN = 64, NMI = WM / 32, NNI = 2;
    static constexpr bool SCALED = std::is_same_v<KIND, FP8>;
    static constexpr int A_STAGE = TM * ROW, STAGE = A_STAGE + TN * ROW, A_LOADS = TM / 32, LOADS = A_LOADS + 4; // direct loads of a thread and step
    static_assert(TM == 128 || TM == 64, "rows of the tile");
    static constexpr int SCALES = 256 * 16;                             // scale bytes of sixteen steps of all rows of a tile
    static constexpr int LDS_BYTES = 4 * STAGE + (SCALED ? 4 * SCALES : 0);
    static constexpr int SUMS = TM * TN * 4;                            // half of the accumulators of all waves
    static constexpr int SR = 16, PITCH = WN * 4 + 16;                  // a wave's strip of the epilogue: 16 rows
    static_assert(SUMS + 8 * SR * PITCH <= LDS_BYTES, "sums and strips fit the stages");
    static constexpr int TILE_FLOATS = TM * TN;
    static constexpr int NK = SCALED ? 2 : 4;
    using FragT = typename PlaneFrag<KIND>::type;
    static_assert(!(KN && SCALED), "FP8 operands are k-contiguous");
    static LCMA_DEV constexpr int swz(int row, int c) { return c ^ ((row >> 1) & 7); }

    struct State {
        __amdgpu_buffer_rsrc_t ra, rb, rs; // rs: the scale bytes that this wave loads, of A or of B
        uint32_t a_voff, a_tail, b_voff, b_tail, a_rows, b_rows, b_step;
        uint32_t a_frag[4], b_frag[4];
        uint32_t s_voff;
        int lane, l32, lh, half, w, wm, wn;
    };
    struct Piece {
        uint32_t a, b, sc; // first byte of the operands (step 0 of the tile-product) and of the scales of this wave's rows
        int y0, y1;        // steps [y0, y1)
    };
    static LCMA_DEV void slot_end() {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    }
    static LCMA_DEV State prepare(const PlaneGemmParams &p) {
        State s;
        const int tid = threadIdx.x, t = tid & 255;
        s.half = __builtin_amdgcn_readfirstlane(tid >> 8);
        s.w = __builtin_amdgcn_readfirstlane(tid >> 6) & 3;
        s.lane = tid & 63;
        s.l32 = tid & 31;
        s.lh = (tid >> 5) & 1;
        s.wm = s.w & 1;
        s.wn = s.w >> 1;
        s.ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.A), 0, (int)p.a_bytes, 0x00020000);
        s.rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.B), 0, (int)p.b_bytes, 0x00020000);
        const int row = t >> 3, c = swz(row, t & 7) * 16;
        s.a_voff = (uint32_t)row * p.lda_b + c;
        s.a_tail = (uint32_t)c < p.tail_b ? s.a_voff : p.a_bytes; // the last step: chunks past K read as zero
        s.a_rows = 32 * p.lda_b;
        if constexpr (KN) { // load q fills rows (k) q * 16 + t / 16, position t % 16, from chunk position ^ 4 (k % 4)
            const int k = t >> 4;
            s.b_tail = s.b_voff = (uint32_t)k * p.ldb_b + ((t & 15) ^ ((k & 3) << 2)) * 16;
            s.b_rows = 16 * p.ldb_b;
            s.b_step = 64 * p.ldb_b;
        } else {
            s.b_voff = (uint32_t)row * p.ldb_b + c;
            s.b_tail = (uint32_t)c < p.tail_b ? s.b_voff : p.b_bytes;
            s.b_rows = 32 * p.ldb_b;
            s.b_step = ROW;
        }
        const int ar = s.wm * WM + s.l32, br = s.wn * WN + s.l32;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int ch = SCALED ? (k >> 1) * 4 + s.lh * 2 + (k & 1) : k * 2 + s.lh;
            s.a_frag[k] = ar * ROW + swz(ar, ch) * 16;
            s.b_frag[k] = br * ROW + swz(br, ch) * 16;
        }
        if constexpr (KN) {
            s.b_frag[0] = column_base(s.lane, s.wn * 2);
            s.b_frag[1] = column_base(s.lane, s.wn * 2 + 1);
        }
        if constexpr (SCALED) {
            // wave w of a group: rows 64 w and on, first those of A, then those of B (TM = 64: the last wave's are nobody's, its load is
            // there for the count)
            const bool of_a = s.w < TM / 64;
            const uint64_t at = of_a ? (uint64_t)p.SA : (uint64_t)p.SB;
            const uint32_t bytes = of_a ? p.sa_bytes : p.sb_bytes, pitch = of_a ? p.lsa_b : p.lsb_b;
            s.s_voff = (uint32_t)(of_a ? t : (t - TM) & 127) * pitch;
            // (uniform anyway; said here so that the descriptor stays in scalar registers)
            const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)at), hi = __builtin_amdgcn_readfirstlane((uint32_t)(at >> 32));
            s.rs = __builtin_amdgcn_make_buffer_rsrc((void *)((uint64_t)hi << 32 | lo), 0, __builtin_amdgcn_readfirstlane(bytes), 0x00020000);
        }
        return s;
    }
    static LCMA_DEV FragT fragment(const LCMA_LDS char *base, const uint32_t (&at)[4], int k) {
        if constexpr (SCALED) {
            const u32x4 lo = *(const LCMA_LDS u32x4 *)(base + at[2 * k]), hi = *(const LCMA_LDS u32x4 *)(base + at[2 * k + 1]);
            return i32x8{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
        } else {
            return __builtin_bit_cast(FragT, *(const LCMA_LDS u32x4 *)(base + at[k]));
        }
    }
    // The steps of a piece: this group's are y0 + half, y0 + half + 2, ...  s0, s1: the group's stages; c0, c1: its scale
    // bytes.
    static LCMA_DEV void steps(const PlaneGemmParams &p, const State &s, const Piece &pc, f32x16 (&acc)[NMI][NNI], LCMA_LDS char *__restrict__ s0,
                               LCMA_LDS char *__restrict__ s1, LCMA_LDS char *__restrict__ c0, LCMA_LDS char *__restrict__ c1) {
        const int ny = p.ny;
        // operands of step y (past the end of the piece: past the extents, zeros); the scalar offsets are uniform anyway, said here
        // so that they stay in scalar registers
        struct Source {
            uint32_t a, b, av, bv;
        };
        auto source = [&](int y) {
            const bool in = y < pc.y1, last = y + 1 == ny;
            return Source{(uint32_t)__builtin_amdgcn_readfirstlane(in ? pc.a + (uint32_t)y * ROW : p.a_bytes), (uint32_t)__builtin_amdgcn_readfirstlane(in ? pc.b + (uint32_t)y * s.b_step : p.b_bytes),
                          last ? s.a_tail : s.a_voff, last ? s.b_tail : s.b_voff};
        };
        auto load_one = [&](LCMA_LDS char *st, const Source &o, int q) {
            if (q < A_LOADS) __builtin_amdgcn_raw_ptr_buffer_load_lds(s.ra, (LCMA_LDS void *)(st + (q * 256 + s.w * 64) * 16), 16, (int)o.av, (int)(o.a + q * s.a_rows), 0, 0);
            else __builtin_amdgcn_raw_ptr_buffer_load_lds(s.rb, (LCMA_LDS void *)(st + A_STAGE + ((q - A_LOADS) * 256 + s.w * 64) * 16), 16, (int)o.bv, (int)(o.b + (q - A_LOADS) * s.b_rows), 0, 0);
        };
        auto load_scales = [&](LCMA_LDS char *to, int step) { // scale bytes of sixteen steps from `step` (a multiple of four) on
            if constexpr (SCALED)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(s.rs, (LCMA_LDS void *)(to + s.w * 64 * 16), 16, (int)s.s_voff, __builtin_amdgcn_readfirstlane(pc.sc + (uint32_t)step), 0, 0);
        };
        // up to two steps are the first group's alone: one chain of sums, the bits of the generated batched kernel
        const int all = pc.y1 - pc.y0, turn = all > 2 ? 2 : 1, n = turn == 2 ? (all + 1) / 2 : all;
        int y = turn == 2 ? pc.y0 + s.half : s.half ? pc.y1 : pc.y0;
        int base = pc.y0 & ~3;
        LCMA_LDS char *cur = c0, *next = c1;
        load_scales(cur, base);
#pragma unroll
        for (int q = 0; q < LOADS; ++q) load_one(s0, source(y), q);
#pragma unroll
        for (int q = 0; q < LOADS; ++q) load_one(s1, source(y + turn), q);
        wait_vm<LOADS>();
        slot_end();
        if (s.half) slot_end(); // the second group runs one slot behind the first
        auto step = [&](LCMA_LDS char *st, auto scales) { // scales: with the load of the next block of scale bytes
            FragT a[NMI][NK], b[NNI][NK];
            int sa[NMI], sb[NNI];
#pragma unroll
            for (int k = 0; k < NK; ++k)
#pragma unroll
                for (int i = 0; i < NMI; ++i) a[i][k] = fragment(st + i * 32 * ROW, s.a_frag, k);
#pragma unroll
            for (int i = 0; i < NNI; ++i) {
                if constexpr (KN) read_columns(st + A_STAGE, s.b_frag[i], b[i]);
                else
#pragma unroll
                    for (int k = 0; k < NK; ++k) b[i][k] = fragment(st + A_STAGE + i * 32 * ROW, s.b_frag, k);
            }
            if constexpr (SCALED) {
                const LCMA_LDS char *at = cur + (y - base);
#pragma unroll
                for (int i = 0; i < NMI; ++i) sa[i] = *(const LCMA_LDS uint8_t *)(at + (s.wm * WM + i * 32 + s.l32) * 16);
#pragma unroll
                for (int i = 0; i < NNI; ++i) sb[i] = *(const LCMA_LDS uint8_t *)(at + (TM + s.wn * WN + i * 32 + s.l32) * 16);
            }
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(0xC07F); // lgkmcnt(0): what was read has left LDS, so behind the barrier its place may be loaded anew
            slot_end();
            if constexpr (SCALED) { // past the end the operands are zeros and the scale bytes nobody's
                if (y >= pc.y1) {
#pragma unroll
                    for (int i = 0; i < NMI; ++i) sa[i] = 127;
#pragma unroll
                    for (int i = 0; i < NNI; ++i) sb[i] = 127;
                }
            }
            const Source o = source(y + 2 * turn);
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int k = 0; k < NK; ++k)
#pragma unroll
                for (int i = 0; i < NMI; ++i) {
#pragma unroll
                    for (int q = (k * NMI + i) * LOADS / (NK * NMI); q < (k * NMI + i + 1) * LOADS / (NK * NMI); ++q) load_one(st, o, q);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int j = 0; j < NNI; ++j) {
                        if constexpr (SCALED) acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a[i][k], b[j][k], acc[i][j], 0, 0, 0, sa[i], 0, sb[j]);
                        else Mma<KIND>::run(a[i][k], b[j][k], acc[i][j]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            __builtin_amdgcn_s_setprio(0);
            if constexpr (SCALED && decltype(scales)::value) { // (behind the loads of the step, so that the wait leaves it in flight)
                load_scales(next, base + 12);
                wait_vm<LOADS + 1>();
            } else {
                wait_vm<LOADS>();
            }
            slot_end();
        };
        // n steps of either group; what lies past the end of the piece is zeros
        for (int i = 0;;) {
#pragma unroll
            for (int j = 0; j < (SCALED ? 6 : 2); ++j) {
                if (j == 0) step(s0, std::true_type());
                else step(j & 1 ? s1 : s0, std::false_type());
                y += turn;
                if (++i == n) goto done;
            }
            if constexpr (SCALED) { // sixteen scale bytes of a row last for twelve steps from any step of their first dword on
                base += 12;
                LCMA_LDS char *t = cur;
                cur = next;
                next = t;
            }
        }
    done:
        wait_vm<0>();
        if (!s.half) slot_end();
    }
    template <int N> static LCMA_DEV void wait_vm() { // all but the N youngest vector memory instructions
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt((N & 15) | (N >> 4) << 14 | 0x0F70);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    }
    // The sums of both groups, each keeping 16 of every 32 rows: of accumulator (i, j) values 8 half to 8 half + 7, i.e. rows 16 half +
    // (v / 4) * 8 + 4 lh + v % 4 of the 32.  (LDS holds nothing that is still needed; a barrier ends it.)
    static LCMA_DEV void add_groups(const State &s, LCMA_LDS char *lds, const f32x16 (&acc)[NMI][NNI], f32x4 (&sum)[NMI][NNI][2]) {
        LCMA_LDS f32x4 *x = (LCMA_LDS f32x4 *)lds;
#pragma unroll
        for (int i = 0; i < NMI; ++i)
#pragma unroll
            for (int j = 0; j < NNI; ++j)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    f32x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = s.half ? acc[i][j][q * 4 + e] : acc[i][j][8 + q * 4 + e];
                    x[(((i * NNI + j) * 2 + q) * 8 + (s.half ^ 1) * 4 + s.w) * 64 + s.lane] = v;
                }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NMI; ++i)
#pragma unroll
            for (int j = 0; j < NNI; ++j)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const f32x4 v = x[(((i * NNI + j) * 2 + q) * 8 + s.half * 4 + s.w) * 64 + s.lane];
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum[i][j][q][e] = v[e] + (s.half ? acc[i][j][8 + q * 4 + e] : acc[i][j][q * 4 + e]);
                }
    }
    // to: the plane of C (or of the partial products), `extent` bytes of rows of `pitch` bytes; row_b: bytes of a row that are written
    template <class T>
    static LCMA_DEV void store_tile(const State &s, LCMA_LDS char *lds, void *to, uint32_t extent, uint32_t pitch, uint32_t row_b, int x, int z, const f32x4 (&sum)[NMI][NNI][2]) {
        constexpr int OES = T::ES, P = WN * OES + 16, CPRW = WN * OES / 16, NIT = SR * CPRW / 64;
        const auto rc = __builtin_amdgcn_make_buffer_rsrc(to, 0, (int)extent, 0x00020000);
        const uint32_t c_base = (uint32_t)x * TM * pitch + (uint32_t)z * TN * OES;
        LCMA_LDS char *strip = lds + SUMS + (s.half * 4 + s.w) * (SR * PITCH);
#pragma unroll
        for (int i = 0; i < NMI; ++i) {
#pragma unroll
            for (int j = 0; j < NNI; ++j)
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        LCMA_LDS char *at = strip + (q * 8 + 4 * s.lh + e) * P + (j * 32 + s.l32) * OES;
                        if constexpr (OES == 2) *(LCMA_LDS uint16_t *)at = (uint16_t)Round<T>::run(sum[i][j][q][e]);
                        else *(LCMA_LDS float *)at = sum[i][j][q][e];
                    }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int it = 0; it < NIT; ++it) {
                const int idx = it * 64 + s.lane, row = idx / CPRW, ch = idx % CPRW;
                const u32x4 v = *(LCMA_LDS u32x4 *)(strip + row * P + ch * 16);
                const uint32_t colb = (uint32_t)(s.wn * WN) * OES + ch * 16;
                const uint32_t off = ((uint32_t)z * TN * OES + colb < row_b) ? c_base + (uint32_t)(s.wm * WM + i * 32 + s.half * 16 + row) * pitch + colb : extent;
                // (16-byte store: the scalar-offset field stays a literal zero, see PlaneGemm::store_tile)
                __builtin_amdgcn_raw_buffer_store_b128(v, rc, (int)off, 0, kStreamed);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
    }
    static LCMA_DEV void store_c(const PlaneGemmParams &p, const State &s, LCMA_LDS char *lds, int plane, int x, int z, const f32x4 (&sum)[NMI][NNI][2]) {
        store_tile<OUT>(s, lds, (char *)p.C + (uint32_t)plane * p.c_plane, p.c_plane ? p.c_plane : p.c_bytes, p.ldc_b, p.n_row_b, x, z, sum);
    }
    static LCMA_DEV Piece piece_of(const PlaneGemmParams &p, const State &s, int plane, int x, int z, int y0, int y1) {
        Piece pc;
        pc.a = (uint32_t)plane * p.a_plane + (uint32_t)(x * TM) * p.lda_b;
        pc.b = (uint32_t)plane * p.b_plane + (KN ? (uint32_t)(z * TN) * 2 : (uint32_t)(z * TN) * p.ldb_b);
        if constexpr (SCALED)
            pc.sc = s.w < TM / 64 ? (uint32_t)plane * p.sa_plane + (uint32_t)(x * TM) * p.lsa_b : (uint32_t)plane * p.sb_plane + (uint32_t)(z * TN) * p.lsb_b;
        pc.y0 = y0;
        pc.y1 = y1;
        return pc;
    }
    static LCMA_DEV void multiply(const PlaneGemmParams &p, const State &s, const Piece &pc, LCMA_LDS char *lds, f32x4 (&sum)[NMI][NNI][2]) {
        f32x16 acc[NMI][NNI];
#pragma unroll
        for (int i = 0; i < NMI; ++i)
#pragma unroll
            for (int j = 0; j < NNI; ++j) zero(acc[i][j]);
        LCMA_LDS char *st = lds + s.half * (2 * STAGE), *sc = lds + (SCALED ? 4 * STAGE + s.half * (2 * SCALES) : 0);
        steps(p, s, pc, acc, st, st + STAGE, sc, sc + (SCALED ? SCALES : 0));
        __syncthreads();
        add_groups(s, lds, acc, sum);
    }
    // one tile-product per work-group; an XCD takes a contiguous run of them
    static LCMA_DEV void run(const PlaneGemmParams &p, LCMA_LDS char *lds) {
        const State s = prepare(p);
        int plane, x, z;
        tile_of_job(p.nx, p.nz, p.panel, eighths(p.jobs), plane, x, z);
        f32x4 sum[NMI][NNI][2];
        multiply(p, s, piece_of(p, s, plane, x, z, 0, p.ny), lds, sum);
        store_c(p, s, lds, plane, x, z, sum);
    }
    static LCMA_DEV int eighths(int n) { // n work-groups: a contiguous eighth of the numbers to every XCD, the rest in turn
        const int per = n >> 3, id = blockIdx.x;
        return id < (per << 3) ? (id & 7) * per + (id >> 3) : id;
    }

    // K in slices of cap steps for work-groups of their own: fp32 partial products, a matrix of whole tiles for every slice, which
    // few_rows_sum adds in ascending order.  Slice by slice, so that work-groups that run side by side share lines.
    static LCMA_DEV void run_slices(const PlaneGemmParams &p, LCMA_LDS char *lds) {
        const State s = prepare(p);
        const int unit = eighths(p.units / 2), slice = unit / p.jobs, y0 = slice * (int)p.cap, y1 = y0 + (int)p.cap < p.ny ? y0 + (int)p.cap : p.ny;
        int plane, x, z;
        tile_of_job(p.nx, p.nz, p.panel, unit - slice * p.jobs, plane, x, z);
        f32x4 sum[NMI][NNI][2];
        multiply(p, s, piece_of(p, s, plane, x, z, y0, y1), lds, sum);
        const uint32_t pitch = p.nz * TN * 4, extent = p.nx * TM * pitch;
        store_tile<F32>(s, lds, (char *)p.partial + (int64_t)slice * extent, extent, pitch, pitch, x, z, sum);
    }

    // Split-Group ranges: work-group u owns steps [u cap, (u + 1) cap), counted through the tile-products.  A whole tile-product
    // among them is stored at once, pieces go to slots (as fp32 sums) for fixup to put together.
    static LCMA_DEV void run_ranges(const PlaneGemmParams &p, LCMA_LDS char *lds) {
        const State s = prepare(p);
        const int ny = p.ny, unit = eighths(p.units);
        const int64_t lo = (int64_t)unit * p.cap, total = (int64_t)p.jobs * ny;
        int job = (int)(lo / ny), y0 = (int)(lo - (int64_t)job * ny);
        int64_t left = p.cap < total - lo ? p.cap : total - lo;
        f32x4 sum[NMI][NNI][2];
        while (left > 0) {
            const int y1 = left < ny - y0 ? y0 + (int)left : ny;
            int plane, x, z;
            tile_of_job(p.nx, p.nz, p.panel, job, plane, x, z);
            multiply(p, s, piece_of(p, s, plane, x, z, y0, y1), lds, sum);
            if (y0 == 0 && y1 == ny) {
                store_c(p, s, lds, plane, x, z, sum);
            } else {
                f32x4 *dst = (f32x4 *)p.partial + (int64_t)(unit * 2 + (y0 == 0)) * (TILE_FLOATS / 4) + threadIdx.x;
#pragma unroll
                for (int i = 0; i < NMI * NNI * 2; ++i) dst[i * NT] = sum[i >> 2][i >> 1 & 1][i & 1];
            }
            left -= y1 - y0;
            ++job;
            y0 = 0;
            __syncthreads(); // (the next loads go where the sums and the strips were)
        }
    }
    // Second kernel of the ranges: one work-group per boundary between work-groups u - 1 and u.  If that boundary is the first one
    // inside its tile-product, adds the pieces of the tile-product in ascending order, rounds once and stores it.
    static LCMA_DEV void fixup(const PlaneGemmParams &p, LCMA_LDS char *lds) {
        const int ny = p.ny, u = blockIdx.x + 1;
        const int64_t total = (int64_t)p.jobs * ny, b = (int64_t)u * p.cap;
        if (b >= total || b % ny == 0) return; // no tile-product straddles this boundary
        const int job = (int)(b / ny);
        if (b - p.cap > (int64_t)job * ny) return; // an earlier boundary lies inside the same tile-product
        const State s = prepare(p);
        f32x4 sum[NMI][NNI][2];
        const f32x4 *src = (const f32x4 *)p.partial + (int64_t)((u - 1) * 2 + 1) * (TILE_FLOATS / 4) + threadIdx.x; // the piece that starts at step 0
#pragma unroll
        for (int i = 0; i < NMI * NNI * 2; ++i) sum[i >> 2][i >> 1 & 1][i & 1] = src[i * NT];
        for (int v = u; (int64_t)v * p.cap < (int64_t)(job + 1) * ny && (int64_t)v * p.cap < total; ++v) {
            src = (const f32x4 *)p.partial + (int64_t)(v * 2) * (TILE_FLOATS / 4) + threadIdx.x;
#pragma unroll
            for (int i = 0; i < NMI * NNI * 2; ++i) sum[i >> 2][i >> 1 & 1][i & 1] += src[i * NT];
        }
        int plane, x, z;
        tile_of_job(p.nx, p.nz, p.panel, job, plane, x, z);
        store_c(p, s, lds, plane, x, z, sum);
    }
};

} // namespace lcma
