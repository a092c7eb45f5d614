// Fused <2,2,2;7> for 16-bit products with few tiles on gfx950: the sibling of lcma_direct.hpp for fp16 and bf16 storage.
//
// The staged kernels give a group of 64 x 64 blocks to one work-group that walks all of K/k in dependent steps of 32: 1000 x 1544 x
// 2056 with <2,2,2;7> is 104 work-groups of 33 steps at 1 us, 239 x 2176 x 9024 is 36 of 141.  Here a group is a tile of 32 x 64
// (or 16 x 64) of every block, a step is 64 k of all of them, and the eight waves of its work-group share the k of a step (and its
// columns; see NW).  Raw blocks in LDS, conversions and sums on the fragments as in the fragment-combine kernels; the partial
// tiles of C are added in LDS, in fp32, always in the same order, and rounded once.  Which k meets which lane is the same for both
// layouts of B, so both give the same bits.  K is padded to multiples of 128, by the staged kernels to 64: where that cuts it elsewhere (2056: 1088
// instead of 1056) other elements of A and of B meet in the sums and are rounded to fp16, so the bits differ from theirs by more than an
// order of sums would make them (8.5e-4 against 4e-5), the error against 64 bits does not (1.67e-3 both).
// Fragments brought from memory straight into registers, as this kernel had them before, take a CU 26 to 64 clocks a load; a
// load with eight lanes to the 128 bytes of a row takes 16.  So raw lines travel straight into LDS, two or three steps ahead
// behind counted waits, and K x N operands are read from there with transposing reads.
// What bounds it: vector instructions (bf16: 224 conversions and sums of 4 clocks per SIMD in a step of the larger tile, against
// 448 clocks of matrix instructions, with which they overlap in part) and the 40 or 48 KB a CU takes in per step, 70 to 80 bytes/ns
// beside the reads from LDS.  Measured (us, before, on 16 x 64 tiles or staged / this; three sets of operands in turn, launches from a graph),
// K x N bf16, N x K bf16, K x N fp16, N x K fp16: 239 x 2176 x 9024 61 / 47, 74 / 48, 54 / 38, 65 / 42; 473 x 344 x 2696 26 / 20, 28 / 21, 23 /
// 19, 25 / 20; 1024^3 15.0 / 10.8, 14.8 / 10.7, 14.1 / 9.6, 15.1 / 9.3; 32 x 64 tiles: 1000 x 1544 x 2056 35.6 / 20.2, 32.6 / 20.0, 31.6 /
// 19.2, 32.5 / 19.3; geometric mean over 280 calls on few tiles 1.39.  Four waves with 32 x 64 tiles each, which convert
// nothing twice: 22 at 1000 x 1544 x 2056 (one wave per SIMD, nothing covers its waits); all waves in step with each other: 21.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lcma_prepare_b.hpp" // for_each_const

namespace lcma {

// IN: storage type.  TM: 32 or 16.  CH, CHH (generated): as for Direct.  TB: B is the N x K matrix W.
template <class IN, int TM, bool TB, class CH, class CHH> struct Direct16 {
    static constexpr int F = TM, TN = 64, NC = CHH::NC;                        // 32x32x16 or 16x16x32 instructions
    // Waves: two groups of four, one wave of each on every SIMD.  32 rows: four along the k of a step, a group to half of the columns; 16
    // rows: two along the k of a step and two along the columns, a group to every second step.
    static constexpr int NW = 8, KW = 4, NI = F == 32 ? 1 : 2, STAGES = F == 32 ? 3 : 4;
    static constexpr int PITCH = TN + 4;                                       // floats
    static constexpr int A_BLOCK = TM * 128, B_BLOCK = 64 * 128, B_AT = CH::NA * A_BLOCK, STAGE = B_AT + CH::NB * B_BLOCK;
    static constexpr int A_LOADS = A_BLOCK / 2048, B_LOADS = B_BLOCK / 2048, LOADS = A_LOADS + B_LOADS; // direct loads of 1 KB of a wave in a step
    static constexpr int SUMS = KW * NC * TM * PITCH * 4, LDS_BYTES = SUMS > STAGES * STAGE ? SUMS : STAGES * STAGE;
    static_assert(2 * CH::NA == NW && 2 * CH::NB == NW, "a wave loads half a block of either operand");
    static_assert((F == 32 || F == 16) && LDS_BYTES <= 160 * 1024, "LDS budget of one CU");
    using Acc = std::conditional_t<F == 32, f32x16, f32x4>;
    static constexpr int NV = F * F / 64;

    // all but the N youngest loads have landed, what this wave read has left LDS, and so for all waves behind the barrier
    template <int N> static LCMA_DEV void step_begin() {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt((N & 15) | (N >> 4) << 14 | 0x0070);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    }

    // Fragments from LDS, of all four blocks of an operand.  Each is one block of instructions that waits for its own results: the
    // compiler would wait for every load in flight in front of its own reads.  K x N operands: two transposing reads of four k;
    // sixteen lanes give the addresses of four rows (k) x 16 columns, four lanes to a row, and get a column each.
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    static LCMA_DEV void read_a_b(uint32_t a, uint32_t b, u32x4 (&fa)[4], u32x4 (&fb)[4]) {
        if constexpr (TB) {
            asm volatile("ds_read_b128 %0, %8\n"
                         "ds_read_b128 %1, %8 offset:%10\n"
                         "ds_read_b128 %2, %8 offset:%11\n"
                         "ds_read_b128 %3, %8 offset:%12\n"
                         "ds_read_b128 %4, %9\n"
                         "ds_read_b128 %5, %9 offset:%13\n"
                         "ds_read_b128 %6, %9 offset:%14\n"
                         "ds_read_b128 %7, %9 offset:%15\n"
                         "s_waitcnt lgkmcnt(0)"
                         : "=&v"(fa[0]), "=&v"(fa[1]), "=&v"(fa[2]), "=&v"(fa[3]), "=&v"(fb[0]), "=&v"(fb[1]), "=&v"(fb[2]), "=&v"(fb[3])
                         : "v"(a), "v"(b), "i"(A_BLOCK), "i"(2 * A_BLOCK), "i"(3 * A_BLOCK), "i"(B_BLOCK), "i"(2 * B_BLOCK), "i"(3 * B_BLOCK)
                         : "memory");
        } else {
            u32x2 r[4][2];
            asm volatile("ds_read_b128 %0, %12\n"
                         "ds_read_b128 %1, %12 offset:%14\n"
                         "ds_read_b128 %2, %12 offset:%15\n"
                         "ds_read_b128 %3, %12 offset:%16\n"
                         "ds_read_b64_tr_b16 %4, %13\n"
                         "ds_read_b64_tr_b16 %5, %13 offset:512\n"
                         "ds_read_b64_tr_b16 %6, %13 offset:%17\n"
                         "ds_read_b64_tr_b16 %7, %13 offset:%18\n"
                         "ds_read_b64_tr_b16 %8, %13 offset:%19\n"
                         "ds_read_b64_tr_b16 %9, %13 offset:%20\n"
                         "ds_read_b64_tr_b16 %10, %13 offset:%21\n"
                         "ds_read_b64_tr_b16 %11, %13 offset:%22\n"
                         "s_waitcnt lgkmcnt(0)"
                         : "=&v"(fa[0]), "=&v"(fa[1]), "=&v"(fa[2]), "=&v"(fa[3]), "=&v"(r[0][0]), "=&v"(r[0][1]), "=&v"(r[1][0]), "=&v"(r[1][1]),
                           "=&v"(r[2][0]), "=&v"(r[2][1]), "=&v"(r[3][0]), "=&v"(r[3][1])
                         : "v"(a), "v"(b), "i"(A_BLOCK), "i"(2 * A_BLOCK), "i"(3 * A_BLOCK), "i"(B_BLOCK), "i"(B_BLOCK + 512), "i"(2 * B_BLOCK),
                           "i"(2 * B_BLOCK + 512), "i"(3 * B_BLOCK), "i"(3 * B_BLOCK + 512)
                         : "memory");
#pragma unroll
            for (int t = 0; t < 4; ++t) fb[t] = u32x4{r[t][0][0], r[t][0][1], r[t][1][0], r[t][1][1]};
        }
    }
    static LCMA_DEV void read_b(uint32_t b, u32x4 (&fb)[4]) {
        if constexpr (TB) {
            asm volatile("ds_read_b128 %0, %4\n"
                         "ds_read_b128 %1, %4 offset:%5\n"
                         "ds_read_b128 %2, %4 offset:%6\n"
                         "ds_read_b128 %3, %4 offset:%7\n"
                         "s_waitcnt lgkmcnt(0)"
                         : "=&v"(fb[0]), "=&v"(fb[1]), "=&v"(fb[2]), "=&v"(fb[3])
                         : "v"(b), "i"(B_BLOCK), "i"(2 * B_BLOCK), "i"(3 * B_BLOCK)
                         : "memory");
        } else {
            u32x2 r[4][2];
            asm volatile("ds_read_b64_tr_b16 %0, %8\n"
                         "ds_read_b64_tr_b16 %1, %8 offset:512\n"
                         "ds_read_b64_tr_b16 %2, %8 offset:%9\n"
                         "ds_read_b64_tr_b16 %3, %8 offset:%10\n"
                         "ds_read_b64_tr_b16 %4, %8 offset:%11\n"
                         "ds_read_b64_tr_b16 %5, %8 offset:%12\n"
                         "ds_read_b64_tr_b16 %6, %8 offset:%13\n"
                         "ds_read_b64_tr_b16 %7, %8 offset:%14\n"
                         "s_waitcnt lgkmcnt(0)"
                         : "=&v"(r[0][0]), "=&v"(r[0][1]), "=&v"(r[1][0]), "=&v"(r[1][1]), "=&v"(r[2][0]), "=&v"(r[2][1]), "=&v"(r[3][0]), "=&v"(r[3][1])
                         : "v"(b), "i"(B_BLOCK), "i"(B_BLOCK + 512), "i"(2 * B_BLOCK), "i"(2 * B_BLOCK + 512), "i"(3 * B_BLOCK), "i"(3 * B_BLOCK + 512)
                         : "memory");
#pragma unroll
            for (int t = 0; t < 4; ++t) fb[t] = u32x4{r[t][0][0], r[t][0][1], r[t][1][0], r[t][1][1]};
        }
    }

    static LCMA_DEV void run(const Params &p, LCMA_LDS char *lds) {
        const int lane = threadIdx.x & 63, r = lane & (F - 1), q = lane / F, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int group = w >> 2, kw = F == 32 ? w & 3 : w & 1, cw = F == 32 ? group : w >> 1 & 1;
        // an eighth of the tiles to every XCD (work-groups go to the eight in turn), cut along the longer side of C, so that the
        // longer operand is read by one XCD only
        const int share = (gridDim.x + 7) / 8, left = gridDim.x % 8, xcd = blockIdx.x % 8;
        const int id = (left && xcd > left ? left * share + (xcd - left) * (share - 1) : xcd * share) + blockIdx.x / 8;
        const bool wide = p.nz * TN >= p.nx * TM;
        const int x = wide ? id % p.nx : id / p.nz, z = wide ? id / p.nx : id % p.nz;
        const auto ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.A), 0, (int)p.a_bytes, 0x00020000);
        const auto rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.B), 0, (int)p.b_bytes, 0x00020000);
        const auto rc = __builtin_amdgcn_make_buffer_rsrc(p.C, 0, (int)p.c_bytes, 0x00020000);
        // The half blocks this wave loads: half u of the rows.  A load brings eight rows of 128 bytes, lanes 8 i ..
        // 8 i + 7 one row.  Rows past M (and, as W, past N) and rows of B past K lie past the extents and read as zero; columns that
        // would alias the next row are sent there: columns of B past N here, columns of A (and W) past K with every load.
        const int u = w & 1;
        uint32_t a_org = 0, a_col = 0, b_org = 0, b_col = 0;
#pragma unroll
        for (int t = 0; t < CH::NA; ++t)
            if (w >> 1 == t) {
                a_col = (uint32_t)CH::a_l(t) * p.a_bcol;
                a_org = (uint32_t)CH::a_i(t) * p.a_brow + (uint32_t)(x * TM) * p.lda_b;
                b_col = TB ? (uint32_t)CH::b_l(t) * p.b_brow : (uint32_t)CH::b_j(t) * p.b_bcol + (uint32_t)(z * TN) * 2; // (TB: b_brow is the byte step along K)
                b_org = TB ? (uint32_t)CH::b_j(t) * p.b_bcol + (uint32_t)(z * TN) * p.ldb_b : (uint32_t)CH::b_l(t) * p.b_brow;
            }
        a_org += (uint32_t)(u * TM / 2) * p.lda_b;
        b_org += (uint32_t)(u * 32) * p.ldb_b;
        // Where 16-byte chunk c of row i sits: k-contiguous rows at c ^ (i / 2 % 8), so that 16 rows at one chunk column meet all banks
        // once; rows of K x N blocks at c ^ 4 (i / 2 % 2) ^ 2 (i / 8 % 2), the same for the four rows x 32 bytes of a transposing read
        // and its neighbours.  Even and odd loads of a block:
        uint32_t av[2], ac[2], bv[2], bc[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            ac[i] = ((lane & 7) ^ (lane >> 4) ^ 4 * (A_LOADS == 1 ? u : i)) * 16;
            av[i] = (uint32_t)(lane >> 3) * p.lda_b + ac[i];
            bc[i] = TB ? ((lane & 7) ^ (lane >> 4) ^ 4 * i) * 16 : ((lane & 7) ^ (lane >> 4 & 1) << 2 ^ i << 1) * 16;
            bv[i] = (uint32_t)(lane >> 3) * p.ldb_b + bc[i];
            if (!TB && b_col + bc[i] >= p.n_row_b) bv[i] = p.b_bytes;
        }
        // The loads of step y (past the last one from the end of the extents: zeros), number i of the wave's into stage st
        uint32_t a_off[2], b_off[2], a_at, b_at;
        auto aim = [&](int y) {
            const bool in = y < p.ny;
            const uint32_t ka = a_col + (uint32_t)y * 128, kb = b_col + (uint32_t)y * 128;
            a_at = in ? a_org + ka : p.a_bytes;
            b_at = in ? b_org + (TB ? kb : b_col + (uint32_t)y * 64 * p.ldb_b) : p.b_bytes;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                a_off[i] = ka + ac[i] < p.k_row_b ? av[i] : p.a_bytes;
                b_off[i] = !TB || kb + bc[i] < p.k_row_b ? bv[i] : p.b_bytes;
            }
        };
        auto load = [&](LCMA_LDS char *st, int i) {
            if (i < A_LOADS)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (LCMA_LDS void *)(st + w * (A_BLOCK / 2) + i * 1024), 16, (int)a_off[i & 1], (int)(a_at + i * 8 * p.lda_b), 0, 0);
            else
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (LCMA_LDS void *)(st + B_AT + w * (B_BLOCK / 2) + (i - A_LOADS) * 1024), 16, (int)b_off[(i - A_LOADS) & 1],
                                                         (int)(b_at + (i - A_LOADS) * 8 * p.ldb_b), 0, 0);
        };
        // this lane's part of the fragments: chunk kc of eight k of a line; rows r of A and columns (cw NI + ni) F + r of B
        const int kc = kw * (F == 32 ? 2 : 4) + q;
        const uint32_t a_frag = r * 128 + (kc ^ (r >> 1 & 7)) * 16;
        uint32_t b_frag[NI];
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
            const int n0 = (cw * NI + ni) * F;
            if constexpr (TB) {
                b_frag[ni] = B_AT + (n0 + r) * 128 + (kc ^ (r >> 1 & 7)) * 16; // (n0: a multiple of 16)
            } else {
                const int i = lane & 15, k = kc * 8 + (i >> 2), c = (n0 + (F == 32 ? lane & 16 : 0)) / 8 + ((i & 3) >> 1);
                b_frag[ni] = B_AT + k * 128 + (c ^ (i >> 3) << 2 ^ (kc & 1) << 1) * 16 + (i & 1) * 8;
            }
        }
        Acc h[CH::NP][1][NI];
        for_each_const<CH::NP>([&](auto s) {
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int v = 0; v < NV; ++v) h[s][0][ni][v] = 0.f;
        });
        auto multiply = [&](const f16x8 (&a)[CH::NP], const f16x8 (&b)[CH::NP], int ni, int from, int to) {
            for_each_const<CH::NP>([&](auto s) {
                if (s < from || s >= to) return;
                if constexpr (F == 32) Mma<F16>::run(a[s], b[s], h[s][0][ni]);
                else h[s][0][ni] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[s], b[s], h[s][0][ni], 0, 0, 0);
            });
        };
#pragma unroll
        for (int y = 0; y < STAGES - 1; ++y) {
            aim(y);
#pragma unroll
            for (int i = 0; i < LOADS; ++i) load(lds + y * STAGE, i);
        }
        // Both groups work half a step (32 rows) or a step apart, so that one wave of a SIMD waits for its fragments while the other
        // converts and adds.  A slot is what lies between two barriers.
        const uint32_t base = (uint32_t)(uintptr_t)lds;
        auto after = [](uint32_t stage) { return stage == (STAGES - 1) * STAGE ? 0u : stage + STAGE; };
        uint32_t now = 0, ahead = (STAGES - 1) * STAGE; // stages read from and loaded into
        u32x4 ar[CH::NA], br[CH::NB];
        f16x8 a[CH::NA], b[CH::NB], ca[CH::NP], cb[CH::NP];
        if constexpr (F == 32) {
            // Two slots to a step; the matrix instructions follow between the conversions of the next step.  Group 0 waits for the
            // stage of a step in front of it, group 1 in the middle of the step before, which is the same barrier.  A stage is
            // read in the first half of a step only, so it may be loaded anew one barrier later.
            constexpr int FIRST = LOADS / 2; // loads of the first slot
            // bf16: group 0 writes the blocks of A back as fp16, in the place it read them from, and group 1 reads them so one slot later
            // (both converting: 1000 x 1544 x 2056 22.4 us, so 21.2).  A loop of its own for each group: the branches on the group inside
            // one loop cost up to a seventh (fp16 239 x 2176 x 9024 on this tile 45 us, so 38).
            constexpr bool SHARE = !std::is_same_v<IN, F16>;
            auto loads = [&](int from, int to) {
#pragma unroll
                for (int i = from; i < to; ++i) load(lds + ahead, i);
                __builtin_amdgcn_sched_barrier(0);
            };
            for_each_const<CH::NP>([&](auto s) { ca[s] = cb[s] = __builtin_bit_cast(f16x8, u32x4{0, 0, 0, 0}); });
            auto steps = [&](auto g) {
                constexpr bool G = decltype(g)::value;
                if constexpr (G) step_begin<LOADS>();
                for (int y = 0; y < p.ny; ++y) {
                    if constexpr (G) step_begin<63>();
                    else step_begin<LOADS>();
                    multiply(ca, cb, 0, 0, 3);
                    aim(y + 2);
                    read_a_b(base + now + a_frag, base + now + b_frag[0], ar, br);
                    loads(0, FIRST);
                    if constexpr (SHARE && !G) {
                        LCMA_LDS char *at = lds + now + a_frag;
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            multiply(ca, cb, 0, 3 + t, 4 + t);
                            a[t] = Convert<IN, F16>::run(ar[t]);
                            *(LCMA_LDS f16x8 *)(at + t * A_BLOCK) = a[t];
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        step_begin<63>();
                        loads(FIRST, LOADS);
#pragma unroll
                        for (int t = 0; t < 4; ++t) b[t] = Convert<IN, F16>::run(br[t]);
                    } else {
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            multiply(ca, cb, 0, 3 + t, 4 + t);
                            a[t] = SHARE ? __builtin_bit_cast(f16x8, ar[t]) : Convert<IN, F16>::run(ar[t]);
                            b[t] = Convert<IN, F16>::run(br[t]);
                            __builtin_amdgcn_sched_barrier(0);
                            if (t == (SHARE ? 1 : 0)) {
                                if constexpr (G) step_begin<FIRST>();
                                else step_begin<63>();
                                loads(FIRST, LOADS);
                            }
                        }
                    }
                    CH::comb_a(a, ca);
                    CH::comb_b(b, cb);
                    now = after(now);
                    ahead = after(ahead);
                }
                if constexpr (!G) step_begin<63>();
            };
            if (group) steps(std::true_type{});
            else steps(std::false_type{});
            multiply(ca, cb, 0, 0, CH::NP);
        } else {
            // A step takes a group two slots, the other group takes the next step one slot later.  A stage is read in one slot, and in
            // the one behind it is loaded anew, three steps ahead.
            auto slot = [&](int y) {
                step_begin<2 * LOADS>();
                aim(y + 3);
#pragma unroll
                for (int i = 0; i < LOADS; ++i) load(lds + ahead, i);
                __builtin_amdgcn_sched_barrier(0);
                ahead = after(ahead);
            };
            now = group * STAGE;
            if (group) slot(0);
            for (int y = group; y < p.ny; y += 2) {
                slot(y);
                u32x4 br1[CH::NB];
                read_a_b(base + now + a_frag, base + now + b_frag[0], ar, br);
                read_b(base + now + b_frag[1], br1);
#pragma unroll
                for (int t = 0; t < 4; ++t) a[t] = Convert<IN, F16>::run(ar[t]);
                CH::comb_a(a, ca);
                __builtin_amdgcn_sched_barrier(0);
                slot(y + 1);
#pragma unroll
                for (int t = 0; t < 4; ++t) b[t] = Convert<IN, F16>::run(br[t]);
                CH::comb_b(b, cb);
                multiply(ca, cb, 0, 0, 3);
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    multiply(ca, cb, 0, 3 + t, 4 + t);
                    b[t] = Convert<IN, F16>::run(br1[t]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                CH::comb_b(b, cb);
                multiply(ca, cb, 1, 0, CH::NP);
                now = after(after(now));
            }
            if ((p.ny - group) % 2 == 0) slot(p.ny);
        }
        step_begin<0>(); // no load is in flight and every wave has read its last fragments: the partial tiles take the place of the stages
        LCMA_LDS float *mine = (LCMA_LDS float *)lds + (F == 32 ? kw : group * 2 + kw) * (NC * TM * PITCH);
        for_each_const<NC>([&](auto o) {
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                const Acc c = CHH::comb(h, o, 0, ni);
#pragma unroll
                for (int v = 0; v < NV; ++v) mine[(o * TM + (v >> 2) * 8 + q * 4 + (v & 3)) * PITCH + (cw * NI + ni) * F + r] = c[v];
            }
        });
        __syncthreads();
        for (int t = threadIdx.x; t < NC * TM * TN / 8; t += 64 * NW) {
            const int col = t % (TN / 8) * 8, row = t / (TN / 8) % TM, o = t / (TN / 8 * TM);
            const LCMA_LDS float *at = (const LCMA_LDS float *)lds + (o * TM + row) * PITCH + col;
            f32x4 sum[2] = {*(const LCMA_LDS f32x4 *)at, *(const LCMA_LDS f32x4 *)(at + 4)};
#pragma unroll
            for (int k = 1; k < KW; ++k)
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
