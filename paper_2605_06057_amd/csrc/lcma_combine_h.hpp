// Stand-alone Combine H for gfx950 (paper Eq. 6; Algorithm 1, stage 4): C_{i,j} = sum_r W[r,i,j] H_r
// with the products H_r read back from memory.  It exists for the unfused dataflow of Algorithm 1,
// which this library provides to be measured against its fused kernels; the fused kernels apply W
// to fp32 accumulators in registers and never run this.
//
// H: R planes of (padded M/m) x (padded N/n) elements in the type the products were written in
// (fp16 or fp32 for 16-bit storage, fp32 for fp32 storage).  The terms are widened to fp32 (exact), added in
// ascending r and the sum is rounded once, to nearest-even, to the storage type of C.  Rows past M
// fall outside the extent of C (dropped by the range check), columns past N are sent there.
//
// HBM-bound: reads R/(m n) and writes 1 element per element of C.  One thread handles one 16-byte
// vector of every plane and writes the m*n vectors it yields, of 8 bytes where the planes hold fp32 and C 16-bit elements.
// (Two 16-byte loads per plane and 16-byte vectors of C there: each load takes every second 16 bytes of its lines and the 25 planes
// of <3,3,3;23> fill 200 registers: 115 us for planes of 2048 x 2048, 4.3 TB/s, now 90, 5.5; 8192 x 14336, <2,2,2;7> 178, now 171.)
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lcma_prepare_b.hpp"

namespace lcma {

// Cache policy of the loads of the planes: for 16-bit C they are read streamed (8192 x 14336, <2,2,2;7> fp16 planes: 109 -> 100 us with a whole
// wave along a row; <4,4,4;49> 164 -> 155; 25 fp32 planes of 2048 x 2048 97 -> 90), except many small ones that the caches hold
// (combine_h_access, host_common.h: <4,4,4;49> 358 x 3840 x 832 as a whole 55 us, streamed 59).  For fp32 C they are not
// (<3,3,3;23> 384^3, weights combined before, 18.4 us, streamed 18.8; 768^3 28.2 / 28.7; <4,4,4;49> 512^3 22.7 / 23.2; from 1000^3 on level).  Many small fp32
// planes of 16-bit C: level (<3,3,3;23> fp16 1340 x 744 x 2464 25.3 / 25.3, 600 x 4096 x 1024 36.0 / 34.9, 768^3 15.4 / 16.4), streamed like the large ones.

// CH (generated): NP planes, NC = m*n outputs with c_i(o), c_j(o); comb(in, o) = Eq. 6 for output o on floats.
// HT: element type of the planes; IN: storage type of C (of the same or of half the size).
template <class IN, class HT, class CH> LCMA_DEV void combine_h_tile(const CombHParams &p) {
    constexpr int ES = IN::ES, HV = HT::ES / ES; // 16 bytes of a plane become 16 / HV bytes of C
    static_assert(HT::ES == ES || (HT::ES == 4 && ES == 2), "planes in the element size of C, or fp32 planes for 16-bit C");
    const auto rh = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.H), 0, (int)p.h_bytes, 0x00020000);
    const auto rc = __builtin_amdgcn_make_buffer_rsrc(p.C, 0, (int)p.c_bytes, 0x00020000);
    // 256 threads: 2^lane_shift vectors of 256 / 2^lane_shift rows; work-groups that start together cover consecutive pieces
    // of the same rows (4 to 24 % faster than consecutive rows of the same piece)
    const uint32_t sh = (uint32_t)p.lane_shift;
    const uint32_t row = blockIdx.y * (256 >> sh) + (threadIdx.x >> sh);
    const uint32_t at = ((blockIdx.x << sh) + (threadIdx.x & ((1u << sh) - 1))) * 16, colb = at / HV; // byte column inside a plane, a block of C
    if (at >= p.h_ld_b || row * p.h_ld_b >= p.h_plane_b) return;
    // the planes stay in registers as loaded and are widened where a sum uses them (see forget_derived)
    u32x4 h[CH::NP];
    auto load = [&](auto policy) {
#pragma unroll
        for (int r = 0; r < CH::NP; ++r)
            h[r] = __builtin_amdgcn_raw_buffer_load_b128(rh, (int)(row * p.h_ld_b + at), (int)(r * p.h_plane_b), decltype(policy)::value);
    };
    if (ES == 2 && (CH::NP <= 16 || p.streamed)) load(std::integral_constant<int, kStreamed>{});
    else load(std::integral_constant<int, 0>{});
    for_each_const<CH::NC>([&](auto oc_) {
        constexpr int o = decltype(oc_)::value;
        // (only where the widened copies of all planes would not fit beside them and the planes themselves do, <4,4,4;49>
        // with 16-bit planes: two waves per SIMD instead of one; with fewer planes the barrier only delays the first sums)
        if constexpr (HV == 1 && CH::NP * 4 > 128 && CH::NP * 4 <= 224) forget_derived(h);
        auto sum = [&](int e) {
            float col[CH::NP];
#pragma unroll
            for (int r = 0; r < CH::NP; ++r) col[r] = Elem<HT>::get(h[r], e);
            return Round<IN>::run(CH::comb(col, o));
        };
        uint32_t v[4 / HV];
#pragma unroll
        for (int e = 0; e < 4 / HV; ++e) {
            if constexpr (ES == 2) v[e] = sum(2 * e) | (sum(2 * e + 1) << 16);
            else v[e] = sum(e);
        }
        const uint32_t cb = (uint32_t)CH::c_j(o) * p.c_bcol + colb;
        const uint32_t off = cb < p.n_row_b ? (uint32_t)CH::c_i(o) * p.c_brow + row * p.ldc_b + cb : p.c_bytes;
        // (stores: the scalar-offset field stays a literal zero, see Ctx::store_c in lcma_device.hpp)
        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
        if constexpr (HV == 1) __builtin_amdgcn_raw_buffer_store_b128(u32x4{v[0], v[1], v[2], v[3]}, rc, (int)off, 0, kStreamed);
        else __builtin_amdgcn_raw_buffer_store_b64(u32x2{v[0], v[1]}, rc, (int)off, 0, kStreamed);
    });
}

} // namespace lcma
