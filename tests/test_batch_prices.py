"""The tiles that Algorithm 1's batched stage and FP8 products take where a price with a step at 5120 tile-products, or one fitted on operands that
stay in the caches, picked a slower kernel; found on the CPU with launchers that only record (tests/host_dispatch.py)."""
import ctypes

import pytest

import host_dispatch as D


def gemm_stage(scheme, dtype, M, N, K):
    status, ran = D.call("lcma_gemm_unfused", ctypes.c_int(1), M, N, K, D.A, K, D.B, N, D.C, N, ctypes.c_int(D.DTYPES[dtype]), D.Scheme(scheme), D.WORK,
                         workspace_bytes(scheme, dtype, M, N, K), ctypes.c_int(1), ctypes.c_void_p(None))
    assert status == 0
    return [x for x in ran if x.startswith("pg_")]


def workspace_bytes(scheme, dtype, M, N, K):
    f = D.lib().lcma_unfused_workspace_bytes
    f.restype = ctypes.c_int64
    return f(*(ctypes.c_int64(x) for x in (M, N, K)), ctypes.c_int(D.DTYPES[dtype]), D.Scheme(scheme).handle)


# whole calls, us: 256 x 256 tiles / 128 x 128 twice to a CU, which was taken
@pytest.mark.parametrize("scheme,dtype,shape", [("laderman", "f16", (9536, 4592, 1584)),    # 329 / 360
                                                ("laderman", "f16", (9832, 2640, 4104)),    # 378 / 418
                                                ("strassen2", "bf16", (5743, 2072, 5288)),  # 253 / 275
                                                ("strassen2", "bf16", (6241, 3080, 7208)),  # 451 / 490
                                                ("strassen2", "bf16", (2402, 8960, 5544)),  # 277 / 300
                                                ("strassen2", "bf16", (2526, 2528, 14032)), # 338 / 365
                                                ("laderman", "bf16", (6404, 2312, 6280)),   # 307 / 332
                                                ("laderman", "f16", (762, 6048, 1032))],    # 45 / 49
                         ids=str)
def test_batches_on_large_tiles(scheme, dtype, shape):
    ran = gemm_stage(scheme, dtype, *shape)
    assert len(ran) == 1 and ran[0].startswith(f"pg_f16_t256_{'f32' if dtype == 'f16' else 'f16'} "), ran


# An odd number of steps, which the ping-pong kernel rounds up; whole calls, us: 256 x 256 a work-group each / in turn / 128 x 128 twice to a CU
@pytest.mark.parametrize("scheme,dtype,shape", [("strassen2", "bf16", (2841, 2576, 1264)),   # 88 / 97 / 94
                                                ("laderman", "f16", (592, 6040, 1688))],     # 59.2 / 62.7 / 68.5
                         ids=str)
def test_odd_steps_a_work_group_each(scheme, dtype, shape):
    ran = gemm_stage(scheme, dtype, *shape)
    assert ran[0].startswith("pg_f16_t256_") and ran[0].endswith(" dealt=0"), ran


# us: 128 x 128 twice to a CU / 256 x 256: many tile-products of few steps keep it
def test_batches_on_small_tiles():
    ran = gemm_stage("strassen2", "bf16", 1536, 1536, 3840)     # 384 x 384 x 960 in 49 planes: 17.9 / 27.8 (the stage)
    assert ran[0].startswith("pg_f16_t128_f16 ") and ran[0].endswith(" dealt=4"), ran


# us: 256 x 256 / what was taken
@pytest.mark.parametrize("shape", [(15346, 5808, 1032),     # 128 / 139 (128 x 128 twice to a CU)
                                   (13080, 1480, 2584),     # 93 / 101 (128 x 128)
                                   (9580, 2168, 12416)],    # 308 / 346 (128 x 128)
                         ids=str)
def test_fp8_on_large_tiles(shape):
    M, N, K = shape
    status, ran = D.call("lcma_fp8_gemm_nt", M, N, K, D.A, D.WORK, D.B, D.WORK + (1 << 36), D.C, N, ctypes.c_void_p(None))
    assert status == 0 and ran[0].startswith("pg_fp8_t256_bf16 "), ran
