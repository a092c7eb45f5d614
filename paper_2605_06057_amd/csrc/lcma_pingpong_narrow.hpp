// The 256 x 128 sibling of the ping-pong plane GEMM (lcma_pingpong.hpp), for products whose 256 x 256 tiles would leave much of
// the chip idle, with the right operand as N x K rows (W) or as the K x N matrix B.  One tile-product per work-group; wave
// tile 64 x 64, the two groups side by side along N; a step is two phases (the upper and the lower 32 rows of the wave tile)
// of eight matrix instructions.  What bounds it is what a CU can pull in (48 KB a step; the matrix instructions take half of
// the step): a phase holds too little to free places early, so the loads go two whole steps ahead into one of three stages
// (144 KB), the count of the wait is the six loads of one step, and the strips of the epilogue reuse the stages.
// Measured (bf16, us): 2048 x 4096 x 14336 210 against 268 for the 256 x 256 tile and 284 for the generated K x N kernel (128 x
// 128 tiles, register staging); 2048 x 4096 x 4096 62 / 81 / 87; 1536^3 19 / 28 / 22; from about one full round of 256 x 256
// tiles on those win (4096^3 132 / 121).
#pragma once
#include "lcma_pingpong.hpp"

namespace lcma {

// KN: the right operand is B, K x N.
template <class KIND, class OUT, bool KN> struct PingPongNarrow {
    static constexpr int TM = 256, TN = 128, NT = 512, ROW = 128, NMI = 2, NNI = 2, WM = 64, WN = 64;
    static constexpr int A_STAGE = TM * ROW, B_STAGE = TN * ROW; // B: 128 rows of 128 bytes, or 64 rows (k) of 256
    static constexpr int LDS_BYTES = 3 * (A_STAGE + B_STAGE);
    static constexpr int SR = 32, PITCH = WN * OUT::ES + 16;
    static_assert(8 * SR * PITCH <= LDS_BYTES, "the strips of all waves fit the stages");
    using FragT = typename PlaneFrag<KIND>::type;
    static LCMA_DEV constexpr int swz(int row, int c) { return c ^ ((row >> 1) & 7); }

    struct State {
        __amdgpu_buffer_rsrc_t ra, rb;
        uint32_t a_voff, a_tail, b_voff, b_tail, a_rows, b_rows; // byte step between the rows of consecutive loads
        uint32_t a_frag[4], b_frag[4];                           // (KN: b_frag[0 .. 1], the wave's two blocks of 32 columns)
        int wave_chunk;
    };
    static LCMA_DEV void slot_end() {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    }
    template <int FROM, int TO> static LCMA_DEV void load(const State &s, __amdgpu_buffer_rsrc_t r, LCMA_LDS char *dst, uint32_t voff, uint32_t off, uint32_t rows) {
#pragma unroll
        for (int q = FROM; q < TO; ++q)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (LCMA_LDS void *)(dst + (q * NT + s.wave_chunk) * 16), 16, (int)voff,
                                                     (int)(off + q * rows), 0, 0);
    }
    static LCMA_DEV void read_a(const State &s, const LCMA_LDS char *st, int mi, FragT (&f)[4]) {
#pragma unroll
        for (int k = 0; k < 4; ++k) f[k] = __builtin_bit_cast(FragT, *(const LCMA_LDS u32x4 *)(st + s.a_frag[k] + mi * 32 * ROW));
    }
    // (KN: with what was read before, this has landed when the function returns)
    static LCMA_DEV void read_b(const State &s, const LCMA_LDS char *st, FragT (&f)[2][4]) {
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) {
            if constexpr (KN) read_columns(st, s.b_frag[ni], f[ni]);
            else
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    f[ni][k] = __builtin_bit_cast(FragT, *(const LCMA_LDS u32x4 *)(st + s.b_frag[k] + ni * 32 * ROW));
        }
    }
    static LCMA_DEV void multiply(const FragT (&a)[4], const FragT (&b)[2][4], f32x16 (&c)[2]) {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            Mma<KIND>::run(a[k], b[0][k], c[0]);
            Mma<KIND>::run(a[k], b[1][k], c[1]);
        }
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_sched_barrier(0);
    }
    static LCMA_DEV void run(const PlaneGemmParams &p, LCMA_LDS char *lds) {
        pipeline(p, lds, lds, lds + A_STAGE, lds + 2 * A_STAGE, lds + 3 * A_STAGE, lds + 3 * A_STAGE + B_STAGE, lds + 3 * A_STAGE + 2 * B_STAGE);
    }
    static LCMA_DEV void pipeline(const PlaneGemmParams &p, LCMA_LDS char *lds, LCMA_LDS char *A0, LCMA_LDS char *A1,
                                  LCMA_LDS char *A2, LCMA_LDS char *B0, LCMA_LDS char *B1,
                                  LCMA_LDS char *B2) {
        State s;
        const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, lh = lane >> 5;
        const int wm = w & 3, wn = w >> 2; // (wn is also the group: waves w and w + 4 share a SIMD)
        s.wave_chunk = w * 64;
        s.ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.A), 0, (int)p.a_bytes, 0x00020000);
        s.rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.B), 0, (int)p.b_bytes, 0x00020000);
        const int ny = p.ny;
        int job = blockIdx.x; // an XCD takes a contiguous run of tile-products
        const int per = p.jobs >> 3;
        if (job < (per << 3)) job = (job & 7) * per + (job >> 3);
        int plane, x, z;
        tile_of_job(p.nx, p.nz, p.panel, job, plane, x, z);
        {
            const int row = tid >> 3, c = swz(row, tid & 7) * 16;
            s.a_voff = (uint32_t)row * p.lda_b + c;
            s.a_tail = (uint32_t)c < p.tail_b ? s.a_voff : p.a_bytes; // the last step: chunks past K read as zero
            s.a_rows = 64 * p.lda_b;
            if constexpr (KN) { // load q fills rows (k) q * 32 + tid / 16, position tid % 16, from chunk position ^ 4 (k % 4)
                const int k = tid >> 4;
                s.b_voff = (uint32_t)k * p.ldb_b + ((tid & 15) ^ ((k & 3) << 2)) * 16;
                s.b_tail = s.b_voff; // rows past K lie past the extent
                s.b_rows = 32 * p.ldb_b;
            } else {
                s.b_voff = (uint32_t)row * p.ldb_b + c;
                s.b_tail = (uint32_t)c < p.tail_b ? s.b_voff : p.b_bytes;
                s.b_rows = 64 * p.ldb_b;
            }
        }
        const int ar = wm * WM + l32, br = wn * WN + l32;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            s.a_frag[k] = ar * ROW + swz(ar, k * 2 + lh) * 16;
            s.b_frag[k] = br * ROW + swz(br, k * 2 + lh) * 16;
        }
        if constexpr (KN) {
            s.b_frag[0] = column_base(lane, wn * 2);
            s.b_frag[1] = column_base(lane, wn * 2 + 1);
        }
        const uint32_t a0 = (uint32_t)plane * p.a_plane + (uint32_t)(x * TM) * p.lda_b;
        const uint32_t b0 = (uint32_t)plane * p.b_plane + (KN ? (uint32_t)(z * TN) * 2 : (uint32_t)(z * TN) * p.ldb_b);
        const uint32_t b_step = KN ? 64 * p.ldb_b : ROW;
        f32x16 acc[NMI][NNI];
#pragma unroll
        for (int mi = 0; mi < NMI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NNI; ++ni) zero(acc[mi][ni]);
        auto a_of = [&](int y) { return y < ny ? a0 + (uint32_t)y * ROW : p.a_bytes; }; // past the end: past the extent
        auto b_of = [&](int y) { return y < ny ? b0 + (uint32_t)y * b_step : p.b_bytes; };
        FragT fa[4], fb[2][4];
        load<0, 4>(s, s.ra, A0, ny == 1 ? s.a_tail : s.a_voff, a_of(0), s.a_rows);
        load<0, 2>(s, s.rb, B0, ny == 1 ? s.b_tail : s.b_voff, b_of(0), s.b_rows);
        load<0, 4>(s, s.ra, A1, ny == 2 ? s.a_tail : s.a_voff, a_of(1), s.a_rows);
        load<0, 2>(s, s.rb, B1, ny == 2 ? s.b_tail : s.b_voff, b_of(1), s.b_rows);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0x0076); // vmcnt(6)
        slot_end();
        if (wn) slot_end(); // the second group runs one slot behind the first
        // one step out of stage (A, B); the loads of two steps on go into (An, Bn), which the step before read
        auto step = [&](LCMA_LDS char *A, LCMA_LDS char *B, LCMA_LDS char *An, LCMA_LDS char *Bn, int y) {
            const uint32_t a2 = a_of(y + 2), b2 = b_of(y + 2);
            const uint32_t av = y + 3 == ny ? s.a_tail : s.a_voff, bv = y + 3 == ny ? s.b_tail : s.b_voff;
            read_a(s, A, 0, fa);
            if constexpr (!KN) read_b(s, B, fb);
            load<0, 3>(s, s.ra, An, av, a2, s.a_rows);
            if constexpr (KN) { // (behind the loads: it waits for its results)
                __builtin_amdgcn_sched_barrier(0);
                read_b(s, B, fb);
            }
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(0xC07F); // lgkmcnt(0)
            slot_end();
            multiply(fa, fb, acc[0]);
            slot_end();
            read_a(s, A, 1, fa);
            load<3, 4>(s, s.ra, An, av, a2, s.a_rows);
            load<0, 2>(s, s.rb, Bn, bv, b2, s.b_rows);
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(0x0076); // vmcnt(6) lgkmcnt(0): the loads of the next step have landed
            slot_end();
            multiply(fa, fb, acc[1]);
            slot_end();
        };
        for (int y = 0;;) {
            step(A0, B0, A2, B2, y);
            if (++y == ny) break;
            step(A1, B1, A0, B0, y);
            if (++y == ny) break;
            step(A2, B2, A1, B1, y);
            if (++y == ny) break;
        }
        if (!wn) slot_end();
        __builtin_amdgcn_s_waitcnt(0x0070);
        slot_end(); // nothing is in flight and every wave has read its last fragments: the stages hold the strips now
        constexpr int OES = OUT::ES, CPRW = WN * OES / 16, NIT = SR * CPRW / 64;
        const uint32_t extent = p.c_plane ? p.c_plane : p.c_bytes;
        const auto rc = __builtin_amdgcn_make_buffer_rsrc((char *)p.C + (uint32_t)plane * p.c_plane, 0, (int)extent, 0x00020000);
        const uint32_t c_base = (uint32_t)x * TM * p.ldc_b + (uint32_t)z * TN * OES;
        LCMA_LDS char *strip = lds + w * (SR * PITCH);
#pragma unroll
        for (int mi = 0; mi < NMI; ++mi) {
#pragma unroll
            for (int ni = 0; ni < NNI; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    LCMA_LDS char *at = strip + ((v >> 2) * 8 + 4 * lh + (v & 3)) * PITCH + (ni * 32 + l32) * OES;
                    if constexpr (OES == 2) *(LCMA_LDS uint16_t *)at = (uint16_t)Round<OUT>::run(acc[mi][ni][v]);
                    else *(LCMA_LDS float *)at = acc[mi][ni][v];
                }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int it = 0; it < NIT; ++it) {
                const int idx = it * 64 + lane, row = idx / CPRW, ch = idx % CPRW;
                const u32x4 v = *(LCMA_LDS u32x4 *)(strip + row * PITCH + ch * 16);
                const uint32_t colb = (uint32_t)(wn * WN) * OES + ch * 16;
                const uint32_t off = ((uint32_t)z * TN * OES + colb < p.n_row_b) ? c_base + (uint32_t)(wm * WM + mi * 32 + row) * p.ldc_b + colb : extent;
                // (16-byte store: the scalar-offset field stays a literal zero, see PlaneGemm::store_tile)
                __builtin_amdgcn_raw_buffer_store_b128(v, rc, (int)off, 0, kStreamed);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
    }
};

} // namespace lcma
