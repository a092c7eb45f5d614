// The 256 x 256 plane GEMM with the two waves of every SIMD in turn ("ping-pong"): same product, operands and argument
// block as PlaneGemm (lcma_plane_gemm.hpp), whole tile-products only, the same bits (every accumulator takes the same
// instructions over the same k in the same order).
//
// What bounds the step of 128 bytes of K: 2048 cycles of matrix instructions per SIMD (two waves, 32 instructions of 32
// cycles each) against 192 KB of fragment reads and 64 KB of direct loads per CU, and the latency of those loads.  In
// PlaneGemm both waves of a SIMD read, multiply and wait at the same time and a load has less than one step to land:
// its matrix pipe is 58 to 66 % busy.  Here
//  - the eight waves are two groups of four, one wave of each on every SIMD, and a step is four phases of two slots: in a
//    slot one group issues memory instructions (the fragment reads of its next eight matrix instructions, one direct load
//    of half an operand tile) while the other group multiplies; a barrier ends every slot and the groups change roles;
//  - the phases are the quadrants of a wave's 128 x 64 tile, A0 B0, A1 B0, A1 B1, A0 B1 (halves of its rows and columns), so
//    a half of an operand tile is read from LDS in ONE phase (half 0 of B a phase early, at the end of the step before,
//    which balances the reads as 8, 8, 4, 4) and its place is free for the load of two steps later in the phase behind;
//  - a load therefore has seven phases (1.75 steps) to land, and the wait for it is a count, vmcnt(12): the six younger
//    pairs of loads stay in flight across the barriers.
// Every direct load goes out two steps ahead of its use, into the next tile-product too, so the pipeline never drains;
// past the last one the loads are sent past the extents (zeros), which keeps the counts.
// Measured, one run, against PlaneGemm's persistent schedule (random operands; in brackets all-zero operands, where the
// chip's power limit does not hide the difference): 8192 x 4096 x 14336 bf16 1182 -> 1393 TFLOP/s (1400 -> 2024);
// 8192 x 14336 x 4096 1212 -> 1382 (1735 -> 2134); 7 planes of 4096 x 7168 x 2048 fp16 1025 -> 1185 (1329 -> 1756); 25
// planes of 2048^3 with fp32 output 847 -> 1002 (1050 -> 1363).  On random operands the matrix pipe alone sustains 1490 to 1570:
// the plain product is at 0.89 of that (pipe 82 % busy), a batch of planes at 0.79 (72 %: a last round that is not full, tiles of 32
// steps); leaving out the stores of C altogether gains 1.5 to 3.5 % more.
// Measured and not kept: a larger count for the waits while the stores of the tile before are in flight (nothing).
#pragma once
#include "lcma_plane_gemm.hpp"

namespace lcma {

// Fragments of 32 columns of a K x N tile in LDS (64 rows of 256 bytes) for the four 32x32x16 instructions of a step: eight k of a
// column are two transposing reads of four.  Sixteen lanes of such a read give the addresses of four rows (k) x 16 columns,
// four lanes to a row, and get a column each; column_base says where.  One block of instructions that waits for its own
// results: the compiler's form of the read carries no alias information and would wait for every load in flight.
// Measured: the K x N kernels run within 1 to 4 % of the N x K ones.
template <class FragT> LCMA_DEV void read_columns(const LCMA_LDS char *tile, uint32_t base, FragT (&f)[4]) {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    u32x2 r[4][2];
    const uint32_t at = (uint32_t)(uintptr_t)tile + base;
    asm volatile("ds_read_b64_tr_b16 %0, %8\n"
                 "ds_read_b64_tr_b16 %1, %8 offset:1024\n"
                 "ds_read_b64_tr_b16 %2, %8 offset:4096\n"
                 "ds_read_b64_tr_b16 %3, %8 offset:5120\n"
                 "ds_read_b64_tr_b16 %4, %8 offset:8192\n"
                 "ds_read_b64_tr_b16 %5, %8 offset:9216\n"
                 "ds_read_b64_tr_b16 %6, %8 offset:12288\n"
                 "ds_read_b64_tr_b16 %7, %8 offset:13312\n"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(r[0][0]), "=&v"(r[0][1]), "=&v"(r[1][0]), "=&v"(r[1][1]), "=&v"(r[2][0]), "=&v"(r[2][1]), "=&v"(r[3][0]), "=&v"(r[3][1])
                 : "v"(at)
                 : "memory");
#pragma unroll
    for (int k = 0; k < 4; ++k) f[k] = __builtin_bit_cast(FragT, u32x4{r[k][0][0], r[k][0][1], r[k][1][0], r[k][1][1]});
}
// Byte of this lane's part of the first read for the 32 columns from 32 `block` on (block: 0 .. 3).  16-byte chunk c of row k sits at
// position c ^ 4 (k % 4): the four rows of a read are 64 bytes apart in the banks.  Lane group lane / 16: columns 16 (group % 2), k 8
// (group / 2).
LCMA_DEV uint32_t column_base(int lane, int block) {
    const int i = lane & 15, g = lane >> 4, k = i >> 2;
    return (uint32_t)(((g >> 1) * 8 + k) * 256 + ((block * 4 + (g & 1) * 2 + ((i & 3) >> 1)) ^ (k << 2)) * 16 + (i & 1) * 8);
}

// KN: the right operand is the K x N matrix B, not the rows of W (16-bit types).  Half h of its tile is 64 rows (k) of 128 columns,
// 128 h and on, and wave column wn holds columns 32 wn .. of both halves; fragments are read with the transposing LDS read.
template <class KIND, class OUT, bool KN = false> struct PingPongGemm {
    static constexpr int TM = 256, TN = 256, NT = 512, WM = 128, WN = 64, NMI = 4, NNI = 2, ROW = 128;
    static constexpr bool SCALED = std::is_same_v<KIND, FP8>;
    // fragments of a step per tile row: FP8 two of 32 bytes, 16-bit four of 16 bytes
    static constexpr int NK = SCALED ? 2 : 4;
    static constexpr int HALF = 128 * ROW; // bytes of half an operand tile: 128 rows
    // strips of the epilogue, private to a wave, beside the stages (which hold the next tile-product by then)
    static constexpr int SR = OUT::ES == 4 ? 8 : 16, PITCH = WN * OUT::ES + 16, STRIP = SR * PITCH;
    static constexpr int SCALES = SCALED ? 2 * NT * 4 : 0; // two groups of a dword per tile row
    static constexpr int LDS_BYTES = 8 * HALF + 8 * STRIP + SCALES;
    static_assert(LDS_BYTES <= 160 * 1024, "LDS budget of one CU");
    using FragT = typename PlaneFrag<KIND>::type;
    static_assert(!(KN && SCALED), "FP8 operands are k-contiguous");
    static constexpr int NI_COLS = KN ? 128 : 32; // columns from a wave's first 32 to its second

    // as in PlaneGemm: 16-byte chunk c of a row sits at position swz(row, c)
    static LCMA_DEV constexpr int swz(int row, int c) { return c ^ ((row >> 1) & 7); }

    struct State {
        __amdgpu_buffer_rsrc_t ra, rb, rs; // rs: the scale bytes this wave loads (first group: of A, second: of B)
        uint32_t a_voff, b_voff;                         // of this thread's chunk in the first 64 rows of half 0
        uint32_t a_tail, b_tail;                         // the same in the last step: past the extents for chunks past K
        uint32_t a_rows, b_rows, a_half, b_half;         // byte step to the other 64 rows of a half, and to half 1
        uint32_t a_frag[4], b_frag[4];
        int wave_chunk, w, wm, wn, l32, lh;
    };

    // The end of a slot.  (Not __syncthreads(): its fences would wait for the loads in flight.  The scheduling barriers keep
    // matrix instructions, which touch no memory, in their slot.)
    static LCMA_DEV void slot_end() {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    }
    // The end of a slot of memory instructions.  lgkmcnt(0): what this wave reads has left LDS, so behind the barrier the place
    // may be loaded anew; vmcnt(12): all but the six youngest pairs of loads have landed, so behind the barrier any wave may
    // read the half tile of the next phase (other vector memory instructions in between only make the wait stricter).
    static LCMA_DEV void memory_slot_end() {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0x007C);
        slot_end();
    }

    // half an operand tile: 128 rows of 128 bytes, two loads per thread
    static LCMA_DEV void load_half(const State &s, __amdgpu_buffer_rsrc_t r, LCMA_LDS char *dst, uint32_t voff, uint32_t off, uint32_t rows) {
#pragma unroll
        for (int q = 0; q < 2; ++q)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (LCMA_LDS void *)(dst + (q * NT + s.wave_chunk) * 16), 16, (int)voff,
                                                     (int)(off + q * rows), 0, 0);
    }
    static LCMA_DEV FragT fragment(const LCMA_LDS char *base, const uint32_t (&at)[4], int k) {
        if constexpr (SCALED) {
            const u32x4 lo = *(const LCMA_LDS u32x4 *)(base + at[2 * k]), hi = *(const LCMA_LDS u32x4 *)(base + at[2 * k + 1]);
            return i32x8{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
        } else {
            return __builtin_bit_cast(FragT, *(const LCMA_LDS u32x4 *)(base + at[k]));
        }
    }
    static LCMA_DEV void read_a(const State &s, const LCMA_LDS char *half, FragT (&f)[2][NK]) {
#pragma unroll
        for (int k = 0; k < NK; ++k)
#pragma unroll
            for (int i = 0; i < 2; ++i) f[i][k] = fragment(half + i * 32 * ROW, s.a_frag, k);
    }
    // (KN: what was read before has landed as well when the function returns)
    static LCMA_DEV void read_b(const State &s, const LCMA_LDS char *half, FragT (&f)[NK]) {
        if constexpr (KN) read_columns(half, s.b_frag[0], f);
        else
#pragma unroll
            for (int k = 0; k < NK; ++k) f[k] = fragment(half, s.b_frag, k);
    }
    // a quadrant: two accumulators, ascending k (the lowest byte of a scale register is the one that counts)
    static LCMA_DEV void multiply(const FragT (&a)[2][NK], const FragT (&b)[NK], f32x16 &c0, f32x16 &c1, int sa0, int sa1, int sb) {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(1); // the multiplying wave of a SIMD issues ahead of the one that sends memory instructions
#pragma unroll
        for (int k = 0; k < NK; ++k) {
            if constexpr (SCALED) {
                c0 = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a[0][k], b[k], c0, 0, 0, 0, sa0, 0, sb);
                c1 = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a[1][k], b[k], c1, 0, 0, 0, sa1, 0, sb);
            } else {
                Mma<KIND>::run(a[0][k], b[k], c0);
                Mma<KIND>::run(a[1][k], b[k], c1);
            }
        }
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_sched_barrier(0);
    }

    // The argument block is read from the kernel's argument segment where it is needed: kept in scalar registers through the
    // steps, its fields push the offsets of the loads out of them (and the compiler then loops over the lanes of each load).
    typedef const __attribute__((address_space(4))) PlaneGemmParams *Args;

    // (the argument block has to be the kernel's first argument)
    static LCMA_DEV void run(LCMA_LDS char *lds) {
        pipeline((Args)__builtin_amdgcn_kernarg_segment_ptr(), lds, lds + HALF, lds + 2 * HALF, lds + 3 * HALF, lds + 4 * HALF, lds + 5 * HALF, lds + 6 * HALF, lds + 7 * HALF,
                 lds + 8 * HALF, lds + 8 * HALF + 8 * STRIP);
    }

    // Ahs, Bhs: half h of the operand tile in stage s.  restrict: the loads in flight towards one of them do not touch what is
    // read from another, without which the compiler waits for all of them in front of every read.
    static LCMA_DEV void pipeline(Args p, LCMA_LDS char *__restrict__ A00, LCMA_LDS char *__restrict__ A10,
                                  LCMA_LDS char *__restrict__ A01, LCMA_LDS char *__restrict__ A11, LCMA_LDS char *__restrict__ B00,
                                  LCMA_LDS char *__restrict__ B10, LCMA_LDS char *__restrict__ B01, LCMA_LDS char *__restrict__ B11,
                                  LCMA_LDS char *__restrict__ strips, LCMA_LDS char *__restrict__ scales) {
        State s;
        const int tid = threadIdx.x;
        s.w = __builtin_amdgcn_readfirstlane(tid >> 6);
        s.wm = s.w >> 2; // (also the group: waves w and w + 4 share a SIMD)
        s.wn = s.w & 3;
        s.l32 = tid & 31;
        s.lh = (tid >> 5) & 1;
        s.wave_chunk = s.w * 64;
        s.ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p->A), 0, (int)p->a_bytes, 0x00020000);
        s.rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p->B), 0, (int)p->b_bytes, 0x00020000);
        s.rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(s.wm ? p->SB : p->SA), 0, (int)(s.wm ? p->sb_bytes : p->sa_bytes), 0x00020000);
        // Half h of A holds rows wm * 128 + h * 64 + 0 .. 63 of both wm, half h of B the columns wn * 64 + h * 32 + 0 .. 31 of
        // all wn; load q of a thread fills row q * 64 + tid / 8, position tid % 8 (the swizzle is its own inverse and the
        // same for both q).
        {
            const int row = tid >> 3, c = swz(row, tid & 7) * 16;
            s.a_voff = (uint32_t)row * p->lda_b + c;
            s.a_rows = 128 * p->lda_b;
            s.a_half = 64 * p->lda_b;
            s.a_tail = (uint32_t)c < p->tail_b ? s.a_voff : p->a_bytes;
            if constexpr (KN) { // load q of a thread fills row (k) q * 32 + tid / 16, position tid % 16; rows past K lie past the extent
                const int k = tid >> 4;
                s.b_tail = s.b_voff = (uint32_t)k * p->ldb_b + ((tid & 15) ^ ((k & 3) << 2)) * 16;
                s.b_rows = 32 * p->ldb_b;
                s.b_half = 256;
            } else {
                s.b_voff = (uint32_t)((row >> 5) * 64 + (row & 31)) * p->ldb_b + c;
                s.b_tail = (uint32_t)c < p->tail_b ? s.b_voff : p->b_bytes;
                s.b_rows = 128 * p->ldb_b;
                s.b_half = 32 * p->ldb_b;
            }
        }
        const int ar = s.wm * 64 + s.l32, br = s.wn * 32 + s.l32;
#pragma unroll
        for (int k = 0; k < 4; ++k) { // (the assignment of k to lanes is PlaneGemm's)
            const int c = SCALED ? (k >> 1) * 4 + s.lh * 2 + (k & 1) : k * 2 + s.lh;
            s.a_frag[k] = ar * ROW + swz(ar, c) * 16;
            s.b_frag[k] = br * ROW + swz(br, c) * 16;
        }
        if constexpr (KN) s.b_frag[0] = column_base(tid & 63, s.wn);
        const uint32_t b_step = KN ? 64 * p->ldb_b : ROW; // byte step of B from one step to the next
        // an odd number of steps is rounded up by one whose operands are past the extents, i.e. zero
        const int ny = p->ny, n2 = (ny + 1) & ~1;
        // the tile-products of this work-group, dealt as in PlaneGemm::run
        const int per = p->units >> 3, xcd_jobs = (p->jobs + 7) >> 3;
        int unit = blockIdx.x;
        if (unit < (per << 3)) unit = (unit & 7) * per + (unit >> 3);
        int job, hi = p->jobs, turn = p->units, whole = p->jobs; // whole: tile-products in whole rounds
        if (p->interleave == 2) {
            turn = per;
            job = (int)(blockIdx.x & 7) * xcd_jobs;
            if (job + xcd_jobs < hi) hi = job + xcd_jobs;
            job += (int)(blockIdx.x >> 3);
        } else {
            if (p->interleave == 1) whole = hi / turn * turn;
            job = unit < whole ? unit : (int)blockIdx.x;
        }
        if (job >= hi) return;
        // first byte of the operands (and of the scale rows this wave loads) of tile-product j; past the last one: past the extents
        auto origin = [&](int j, uint32_t &a, uint32_t &b, uint32_t &sc) {
            Args q = p;
            asm volatile("" : "+s"(q));
            a = q->a_bytes;
            b = q->b_bytes;
            sc = SCALED ? (s.wm ? q->sb_bytes : q->sa_bytes) : 0;
            if (j < hi) {
                int plane, x, z;
                tile_of_job(q->nx, q->nz, q->panel, j, plane, x, z);
                a = (uint32_t)plane * q->a_plane + (uint32_t)(x * TM) * q->lda_b;
                b = (uint32_t)plane * q->b_plane + (uint32_t)(z * TN) * (KN ? 2 : q->ldb_b);
                if constexpr (SCALED)
                    sc = s.wm ? (uint32_t)plane * q->sb_plane + (uint32_t)(z * TN) * q->lsb_b
                              : (uint32_t)plane * q->sa_plane + (uint32_t)(x * TM) * q->lsa_b;
            }
            // (uniform anyway; said here so that the offsets that derive from them stay in scalar registers)
            a = __builtin_amdgcn_readfirstlane(a);
            b = __builtin_amdgcn_readfirstlane(b);
            if constexpr (SCALED) sc = __builtin_amdgcn_readfirstlane(sc);
        };
        // Scale bytes: a dword holds four steps of a row.  The dwords of a group of four steps travel into LDS four steps ahead
        // (thread t: tile row t of A, or t - 256 of B) and every lane keeps those of its six rows, shifted down step by step->
        const uint32_t s_voff = SCALED ? (uint32_t)(tid & 255) * (s.wm ? p->lsb_b : p->lsa_b) : 0;
        int group = 0; // which half of the scale buffer holds the coming group
        uint32_t sa[NMI], sb[NNI];
        auto load_scales = [&](uint32_t off, int into) {
            if constexpr (SCALED)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(s.rs, (LCMA_LDS void *)(scales + (into * NT + s.wave_chunk) * 4), 4, (int)s_voff,
                                                         (int)off, 0, 0);
        };
        const uint32_t a_none = p->a_bytes, b_none = p->b_bytes;
        uint32_t a_cur, b_cur, s_cur, a_nxt, b_nxt, s_nxt;
        origin(job, a_cur, b_cur, s_cur);
        FragT fa0[2][NK], fa1[2][NK], fb0[NK], fb1[NK];
        f32x16 acc[NMI][NNI];
        auto load_step = [&](LCMA_LDS char *A0, LCMA_LDS char *A1, LCMA_LDS char *B0, LCMA_LDS char *B1, uint32_t a, uint32_t b, bool last) {
            const uint32_t av = last ? s.a_tail : s.a_voff, bv = last ? s.b_tail : s.b_voff;
            load_half(s, s.rb, B0, bv, b, s.b_rows);
            load_half(s, s.ra, A0, av, a, s.a_rows);
            load_half(s, s.ra, A1, av, a + s.a_half, s.a_rows);
            load_half(s, s.rb, B1, bv, b + s.b_half, s.b_rows);
        };
        load_scales(s_cur, 0);
        load_step(A00, A10, B00, B10, a_cur, b_cur, ny == 1);
        load_step(A01, A11, B01, B11, ny > 1 ? a_cur + ROW : a_none, ny > 1 ? b_cur + b_step : b_none, ny == 2);
        memory_slot_end();
        // A slot of its own, for all waves: the first load of the first step, sent by group 0, goes to the place that both groups read
        // here.  (In the steps the slot of either group that reads half 0 of B has ended when its place is loaded anew.)
        read_b(s, B00, fb0);
        memory_slot_end();
        if (s.wm) slot_end(); // the second group runs one slot behind the first
        // One step out of stage (A0, A1, B0, B1); nextB0: half 0 of B of the next step; a, b: the operands two steps on, which go
        // into this stage (last: they are those of a last step).  The slot of the last multiplication is ended by the caller.
        auto step = [&](LCMA_LDS char *A0, LCMA_LDS char *A1, LCMA_LDS char *B0, LCMA_LDS char *B1, LCMA_LDS char *nextB0, uint32_t a, uint32_t b,
                        bool last) {
            const uint32_t av = last ? s.a_tail : s.a_voff, bv = last ? s.b_tail : s.b_voff;
            read_a(s, A0, fa0);
            load_half(s, s.rb, B0, bv, b, s.b_rows);
            memory_slot_end();
            multiply(fa0, fb0, acc[0][0], acc[1][0], (int)sa[0], (int)sa[1], (int)sb[0]);
            slot_end();
            read_a(s, A1, fa1);
            load_half(s, s.ra, A0, av, a, s.a_rows);
            memory_slot_end();
            multiply(fa1, fb0, acc[2][0], acc[3][0], (int)sa[2], (int)sa[3], (int)sb[0]);
            slot_end();
            if constexpr (!KN) read_b(s, B1, fb1); // (KN: behind the loads, it waits for its results)
            load_half(s, s.ra, A1, av, a + s.a_half, s.a_rows);
            if constexpr (KN) read_b(s, B1, fb1);
            memory_slot_end();
            multiply(fa1, fb1, acc[2][1], acc[3][1], (int)sa[2], (int)sa[3], (int)sb[1]);
            slot_end();
            if constexpr (!KN) read_b(s, nextB0, fb0);
            load_half(s, s.rb, B1, bv, b + s.b_half, s.b_rows);
            if constexpr (KN) read_b(s, nextB0, fb0);
            memory_slot_end();
            multiply(fa0, fb1, acc[0][1], acc[1][1], (int)sa[0], (int)sa[1], (int)sb[1]);
        };
        while (true) {
            int next = job + turn; // (the last, partial round of dealing 1 goes to the work-groups in launch order)
            if (next >= whole && job < whole && whole < hi) next = whole + (int)blockIdx.x;
            origin(next, a_nxt, b_nxt, s_nxt);
#pragma unroll
            for (int mi = 0; mi < NMI; ++mi)
#pragma unroll
                for (int ni = 0; ni < NNI; ++ni) zero(acc[mi][ni]);
            for (int y = 0;;) {
                if constexpr (SCALED) {
                    if ((y & 3) == 0) { // the scales of four steps, and the loads of those of the next four
                        const LCMA_LDS char *g = scales + group * (NT * 4);
#pragma unroll
                        for (int mi = 0; mi < NMI; ++mi) sa[mi] = *(const LCMA_LDS uint32_t *)(g + (s.wm * WM + mi * 32 + s.l32) * 4);
#pragma unroll
                        for (int ni = 0; ni < NNI; ++ni) sb[ni] = *(const LCMA_LDS uint32_t *)(g + (TM + s.wn * WN + ni * 32 + s.l32) * 4);
                        group ^= 1;
                        load_scales(y + 4 < ny ? s_cur + y + 4 : s_nxt, group);
                    }
                }
                const bool in = y + 2 < n2, pad = y + 3 == ny;
                const uint32_t a2 = in ? a_cur + (uint32_t)(y + 2) * ROW : a_nxt, b2 = in ? b_cur + (uint32_t)(y + 2) * b_step : b_nxt;
                const bool none = in ? pad : ny == 1;
                step(A00, A10, B00, B10, B01, a2, b2, (in ? y + 3 : 1) == ny);
                slot_end();
                if constexpr (SCALED) {
                    // (past the last step the scale bytes are nobody's: 1 for the zeros of a rounded-up step)
                    const bool past = y + 1 == ny;
#pragma unroll
                    for (int mi = 0; mi < NMI; ++mi) sa[mi] = past ? 127u : sa[mi] >> 8;
#pragma unroll
                    for (int ni = 0; ni < NNI; ++ni) sb[ni] = past ? 127u : sb[ni] >> 8;
                }
                step(A01, A11, B01, B11, B00, none ? a_none : a2 + ROW, none ? b_none : b2 + b_step, (in ? y + 4 : 2) == ny);
                if constexpr (SCALED) {
#pragma unroll
                    for (int mi = 0; mi < NMI; ++mi) sa[mi] >>= 8;
#pragma unroll
                    for (int ni = 0; ni < NNI; ++ni) sb[ni] >>= 8;
                }
                y += 2;
                if (y >= n2) break;
                slot_end();
            }
            // both groups write their halves of the tile in one slot: the first ends the slot of its last multiplication
            // before, the second after
            if (!s.wm) slot_end();
            // the loads past the end have landed before the LDS they go to can be another work-group's (here they are the only
            // ones in flight; behind the stores the wait would be for those too)
            if (next >= hi) __builtin_amdgcn_s_waitcnt(0x0070);
            store_tile(p, s, strips, job, acc);
            if (s.wm) slot_end();
            if (next >= hi) break;
            job = next;
            a_cur = a_nxt;
            b_cur = b_nxt;
            s_cur = s_nxt;
        }
        if (!s.wm) slot_end();
    }

    // As PlaneGemm::store_tile (16-bit C through strips in LDS as whole lines, no barrier), in strips of SR rows.
    static LCMA_DEV void store_tile(Args p, const State &s, LCMA_LDS char *lds, int job, const f32x16 (&acc)[NMI][NNI]) {
        constexpr int OES = OUT::ES, CPRW = WN * OES / 16, NIT = SR * CPRW / 64;
        asm volatile("" : "+s"(p));
        int plane, x, z;
        tile_of_job(p->nx, p->nz, p->panel, job, plane, x, z);
        // batched: the extent is that of the plane, so a tile may hang over the end of it (what it reads there is the next
        // plane's and goes into rows that are dropped here)
        const uint32_t extent = p->c_plane ? p->c_plane : p->c_bytes;
        const auto rc = __builtin_amdgcn_make_buffer_rsrc((char *)p->C + (uint32_t)plane * p->c_plane, 0, (int)extent, 0x00020000);
        const uint32_t c_base = (uint32_t)x * TM * p->ldc_b + (uint32_t)z * TN * OES;
        LCMA_LDS char *strip = lds + s.w * STRIP;
        // (the lane number anew, hidden: what derives from it would otherwise be kept in registers through the steps)
        int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        asm volatile("" : "+v"(lane));
        const int l32 = lane & 31, lh = lane >> 5;
#pragma unroll
        for (int mi = 0; mi < NMI; ++mi) {
#pragma unroll
            for (int h = 0; h < 32 / SR; ++h) {
#pragma unroll
                for (int ni = 0; ni < NNI; ++ni)
#pragma unroll
                    for (int v = h * (SR / 2); v < (h + 1) * (SR / 2); ++v) {
                        LCMA_LDS char *at = strip + ((v >> 2) * 8 + 4 * lh + (v & 3) - h * SR) * PITCH + (ni * 32 + l32) * OES;
                        if constexpr (OES == 2) *(LCMA_LDS uint16_t *)at = (uint16_t)Round<OUT>::run(acc[mi][ni][v]);
                        else *(LCMA_LDS float *)at = acc[mi][ni][v];
                    }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); // (for the compiler: the reads stay behind the writes)
#pragma unroll
                for (int it = 0; it < NIT; ++it) {
                    const int idx = it * 64 + lane, row = idx / CPRW, ch = idx % CPRW;
                    const u32x4 v = *(LCMA_LDS u32x4 *)(strip + row * PITCH + ch * 16);
                    // byte column inside the tile (2 OES chunks of 16 bytes are 32 columns)
                    const uint32_t colb = (uint32_t)(s.wn * (KN ? 32 : WN) + ch / (2 * OES) * NI_COLS) * OES + ch % (2 * OES) * 16;
                    const uint32_t off = ((uint32_t)z * TN * OES + colb < p->n_row_b)
                                             ? c_base + (uint32_t)(s.wm * WM + mi * 32 + h * SR + row) * p->ldc_b + colb
                                             : extent;
                    // (16-byte store: the scalar-offset field stays a literal zero, see PlaneGemm::store_tile)
                    __builtin_amdgcn_raw_buffer_store_b128(v, rc, (int)off, 0, kStreamed);
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            }
        }
    }
};

} // namespace lcma
