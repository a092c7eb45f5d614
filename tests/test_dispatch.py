"""Which kernel a call takes, on the host: the library's own dispatch with launchers that only record (tests/host_dispatch.py)."""
import ctypes

import pytest

import host_dispatch as D

GIB2 = 1 << 31


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("nk", [False, True], ids=["KxN", "NxK"])
def test_a_direct_kernel_refuses_nothing(dtype, nk):
    # spans just below 2 GiB on the staged kernel, which pads K to 64; the direct one pads it to 128 and would reach the limit
    M, N, K = 16, 128, (1 << 23) - 64
    status, ran = D.gemm(M, N, K, dtype, "strassen", nk)
    assert status == 0, D.lib().lcma_last_error()
    assert len(ran) == 1 and ran[0].startswith(f"strassen_{dtype}_t64x64x32"), ran
    assert D.gemm(M, N, K - (1 << 22), dtype, "strassen", nk)[1][0].startswith(f"strassen_{dtype}_d16x64k4")  # (its usual kernel)
    status, ran = D.gemm(M, N, K + 64, dtype, "strassen", nk)   # what was too large stays so
    assert (status, ran) == (5, [])


# A round of 256 work-groups of the 32 x 32 tile and a few more, and a short K: the smaller tile is the faster one, the larger one slower
# than the staged kernel (measured, csrc/api.cc); prepared operands have N padded to whole 64 columns of every block.
@pytest.mark.parametrize("scheme", ["strassen", "winograd"])
def test_small_fp32_products_take_the_smaller_tile(scheme):
    M, N, K = 848, 1388, 192
    for ran in (D.gemm(M, N, K, "f32", scheme), D.gemm(M, N, K, "f32", scheme, True), D.gemm_prepared(M, N, K, "f32", scheme)):
        assert ran[0] == 0 and ran[1][0].startswith(f"{scheme}_f32_d16x16k8"), ran
    assert D.gemm_prepared(1614, 572, 128, "f32", scheme) == (0, [f"{scheme}_f32_d16x16k8b"])
    assert D.gemm(1614, 572, 128, "f32", scheme) == (0, [f"{scheme}_f32_d32x32k8"])   # (234 work-groups: one round)


def test_nt_ws_leaves_a_small_workspace_alone():
    """include/lcma.h: half of lcma_split_group_scratch_bytes() serves the ranges on 128 x 128 tiles alone, fewer bytes nothing."""
    whole = D.lib().lcma_split_group_scratch_bytes()
    for M, N, K in ((64, 4096, 14336), (755, 96, 10368), (512, 4096, 14336)):
        split, none = D.gemm_nt_ws(M, N, K, "bf16", whole), D.gemm_nt_ws(M, N, K, "bf16", 0)
        assert split[0] == 0 and split != none
        for few in (4 << 20, whole // 2 - 256):
            assert D.gemm_nt_ws(M, N, K, "bf16", few) == none
        for half in (whole // 2, whole - 256):
            ran = D.gemm_nt_ws(M, N, K, "bf16", half)[1]
            assert len(ran) == 1 and ("slices=1" in ran[0] or "few_rows" not in ran[0]), ran
        assert none[0] == 0 and len(none[1]) == 1 and ("slices=1" in none[1][0] or "few_rows" not in none[1][0]), none
    # 128 tiles of 224 steps in ranges (92 us)
    assert D.gemm_nt_ws(512, 4096, 14336, "bf16", whole // 2)[1][0].startswith("pg_bf16_t128_bf16 jobs=128 units=512 ")


# Measured (us; weights combined before): plain 62.4, 206, 403, 703, 6606; Algorithm 1 with <2,2,2;7> 71.7, 265, 393, 819, 6270, with <4,4,4;49>
# 86, 304, 427, 854, 6009
@pytest.mark.parametrize("shape,want", [((2048, 4096, 4096), (0, 0)), ((8192, 4096, 4096), (0, 0)), ((6144, 6144, 6144), (1, 1)),
                                        ((8192, 14336, 4096), (0, 0)), ((16384, 16384, 16384), (2, 1))], ids=str)
def test_select_dataflow_prices_all_forms_by_the_present_kernels(shape, want):
    from paper_2605_06057_amd import binding as B
    c = B.lcma_select_dataflow(*shape, B.LCMA_BF16, True)
    assert (c["scheme_id"], c["dataflow"]) == want
    published = B.lcma_predict_unfused_seconds if want[1] else lambda i, M, N, K, dt, _: B.lcma_predict_seconds(i, M, N, K, dt)
    assert c["seconds"] == published(want[0], *shape, B.LCMA_BF16, True)


# Measured, us, generated kernel / 256 x 128 ping-pong kernel: 4.5 / 6.9, 3.5 / 5.7, 6.5 / 9.0, 10.4 / 12.6; the last with rows that do not start on
# lines, 104 / 130 (256 x 256: 168)
@pytest.mark.parametrize("shape,ld", [((839, 1400, 192), 0), ((136, 5488, 64), 0), ((2210, 512, 512), 0), ((942, 1160, 832), 0), ((1178, 2592, 9952), 8)], ids=str)
def test_plain_products_that_the_generated_kernel_does_faster(shape, ld):
    for dtype in ("bf16", "f16"):
        status, ran = D.gemm(*shape, dtype, None, True, ld)
        assert status == 0 and ran[0].startswith(f"plain_{dtype}_t"), ran
        for tall in ((5913, 472, 8776), (7153, 328, 8192)):   # (K x N: 145 / 175, 105 / 121)
            status, ran = D.gemm(*tall, dtype)
            assert status == 0 and ran[0].startswith(f"plain_{dtype}_t"), ran


# Measured, us, a work-group per 128 x 128 tile / what was taken: 91 / 112 (ranges of steps; 256 x 128 ping-pong 86), 143 / 189 (ping-pong 117),
# 14.4 / 15.7 and 9.2 / 10.4 (256 x 128 ping-pong)
def test_nt_ws_between_the_plane_gemm_and_its_kin():
    whole = D.lib().lcma_split_group_scratch_bytes()
    for shape, pad in (((857, 3720, 7040), 8), ((559, 7184, 9856), 0)):
        ran = D.gemm_nt_ws(*shape, "f16", whole, shape[2] + pad)[1]
        jobs, units = (int(ran[0].split(k + "=")[1].split()[0]) for k in ("jobs", "units"))
        assert len(ran) == 1 and units == min(jobs, 256 if "t128" not in ran[0] else 512), ran   # no ranges
    for shape, pad in (((840, 5592, 768), 64), ((4358, 256, 640), 64)):
        assert D.gemm_nt_ws(*shape, "bf16", whole, shape[2] + pad)[1][0].startswith("pg_bf16_t128_bf16 ")
    ran = D.gemm_nt_ws(512, 4096, 14336, "bf16", whole)[1]   # 128 tiles of 224 steps: ranges, 95 us against 221
    assert ran[0].startswith("pg_bf16_t128_bf16 jobs=128 units=512 "), ran


# Measured, us, the fastest other form / what is taken: in four slices 13.3 / 9.1, 40 (128 x 128 tiles) / 28 and 28.5 and 29.5, 8.0 (128 x 128 tiles) / 5.3,
# 31 / 16.6, 32 / 22 (ranges of steps), 12.3 (64 x 64 tiles in two slices) / 9.6; in one piece 39 (tiles of 32) / 30, 20.5 / 16.9
@pytest.mark.parametrize("shape,tile,slices", [((64, 4096, 4096), 32, 1), ((320, 4096, 4096), 64, 1), ((400, 4096, 4096), 64, 1), ((512, 4096, 4096), 64, 1), ((109, 2432, 640), 32, 1),
                                               ((4266, 128, 4288), 64, 1), ((2372, 256, 6656), 64, 1), ((250, 2000, 2112), 32, 1), ((64, 4096, 14336), 64, 4), ((250, 2000, 6400), 64, 2)], ids=str)
def test_few_rows_are_priced_by_the_present_kernels(shape, tile, slices):
    whole = D.lib().lcma_split_group_scratch_bytes()
    for dtype in ("bf16", "f16"):
        ran = D.gemm_nt_ws(*shape, dtype, whole)[1]
        assert ran[0].startswith(f"few_rows_{dtype}_{tile} ") and f" slices={slices} " in ran[0], ran


# What a few-rows kernel would take longer for: 1753 x 2000 x 7552 124 us, here 69 (ping-pong); 2506 x 1056 x 4288 49 / 41; 512 x 4096 x 14336 109 / 92 (ranges of steps)
@pytest.mark.parametrize("shape", [(1753, 2000, 7552), (2506, 1056, 4288), (1292, 1920, 7488), (421, 6656, 2176), (512, 4096, 14336), (512, 4096, 12288)], ids=str)
def test_many_tiles_are_not_few_rows(shape):
    assert "few_rows" not in D.gemm_nt_ws(*shape, "bf16", D.lib().lcma_split_group_scratch_bytes())[1][0]


# Measured, us, four waves with two lines in flight each / eight with four (one work-group per CU): 3.9 / 6.0, 7.6 / 12.1, 26.0 / 30.4, 3.7 / 4.3, 25.6 / 22.5
@pytest.mark.parametrize("shape,deep", [((16, 8192, 512), 0), ((1, 14336, 1024), 0), ((16, 14336, 4096), 0), ((1, 1000, 2048), 0), ((1, 4096, 14336), 1)], ids=str)
def test_few_rows_wait_with_as_many_work_groups_as_fit(shape, deep):
    for space in (0, D.lib().lcma_split_group_scratch_bytes()):
        ran = D.gemm_nt_ws(*shape, "bf16", space)[1]
        assert ran[0].startswith("few_rows_bf16_16 ") and ran[0].endswith(f" deep={deep}"), ran


# Combine H, lanes along a row and cache policy: many small fp16 planes 7.9 us with 16 lanes, 10.5 with 64 and streamed loads (<4,4,4;49>, planes
# of 128 x 1024)
@pytest.mark.parametrize("scheme,shape,lanes", [("strassen2", (358, 3840, 832), 16), ("laderman", (1340, 744, 2464), 16), ("strassen", (2048, 4096, 4096), 64),
                                                ("strassen", (8192, 14336, 4096), 64)], ids=str)
def test_combine_h_access(scheme, shape, lanes):
    M, N, K = shape
    status, ran = D.call("lcma_gemm_unfused", ctypes.c_int(1), M, N, K, D.A, K, D.B, N, D.C, N, ctypes.c_int(D.DTYPES["bf16"]), D.Scheme(scheme), D.WORK,
                         1 << 40, ctypes.c_int(0), ctypes.c_void_p(None))
    assert status == 0 and ran[-1] == f"comb_h_{scheme}_bf16 lanes={lanes} streamed={int(lanes == 64)}"


# ------------------------------------------------------------------ the GPU tests of these kernels reach them
def gemm_on_lines(M, N, K, dtype, nk):
    import test_gpu_plain_pingpong as T
    return D.call("lcma_gemm_nt" if nk else "lcma_gemm", M, N, K, D.A, T.pitch(K), D.B, T.pitch(K if nk else N), D.C, N + 8,
                  ctypes.c_int(D.DTYPES[dtype]), ctypes.c_void_p(None), ctypes.c_void_p(None))


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_shapes_of_the_plain_ping_pong_tests(dtype):
    import test_gpu_plain_pingpong as T
    for shape in T.SHAPES:
        names = ((f"ppn_{dtype}_kn", f"ppn_{dtype}") if shape in T.NARROW else (f"pp_kn_{dtype}", f"pg_{dtype}_t256_{dtype}"))
        for nk in (False, True):
            status, ran = gemm_on_lines(*shape, dtype, nk)
            assert status == 0 and len(ran) == 1, ran
            assert (ran[0].split()[0] == names[nk]) != (nk and shape in T.KN_ONLY), (shape, nk, ran)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_shapes_of_the_few_rows_tests(dtype):
    import test_gpu_few_rows as T
    whole = D.lib().lcma_split_group_scratch_bytes()
    for (M, N, K), plans in T.PLANS.items():
        for (tile, slices), space in zip(plans, (whole, 0)):
            for lda in (K, K + 8):
                status, ran = D.gemm_nt_ws(M, N, K, dtype, space, lda)
                assert status == 0 and len(ran) == 1 + (slices > 1), ran
                assert ran[0].startswith(f"few_rows_{dtype}_{tile} ") and f" slices={slices} " in ran[0], ran


def test_shapes_of_the_direct_tests():
    import test_gpu_direct as F
    import test_gpu_direct16 as H
    for scheme in ("strassen", "winograd"):
        for shape in F.SHAPES[1:]:
            tile = "d32x32k8" if shape == (857, 1048, 808) else "d16x16k8"
            for nk in (False, True):
                assert D.gemm(*shape, "f32", scheme, nk) == (0, [f"{scheme}_f32_{tile}" + "t" * nk])
    for dtype in ("bf16", "f16"):
        for shape in H.CHOSEN:
            for nk in (False, True):
                assert D.gemm(*shape, dtype, "strassen", nk) == (0, [f"strassen_{dtype}_d16x64k4" + "t" * nk])
