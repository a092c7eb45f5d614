"""The kernel that lcma_gemm_nt_ws takes where prices measured on one hot set of operands, or with one penalty for rows off lines whichever
operand has them, picked a slower one; found on the CPU with launchers that only record (tests/host_dispatch.py)."""
import ctypes

import pytest

import host_dispatch as D


def first_launch(M, N, K, pad_a=0, pad_w=0, workspace=True):
    whole = D.lib().lcma_split_group_scratch_bytes()
    status, ran = D.call("lcma_gemm_nt_ws", M, N, K, D.A, K + pad_a, D.B, K + pad_w, D.C, N, ctypes.c_int(D.DTYPES["bf16"]), D.WORK if workspace else 0,
                         whole if workspace else 0, ctypes.c_void_p(None))
    assert status == 0
    return ran[0]


# Tiles of 16: eight waves with four lines in flight each, us: as now / with four waves and two lines (three sets of operands in turn)
@pytest.mark.parametrize("shape", [(1, 1096, 11840),    # 8.2 / 11.1
                                   (1, 920, 9664),      # 7.2 / 9.3
                                   (2, 928, 8832),      # 6.9 / 8.8
                                   (2, 728, 10112),     # 7.6 / 9.7
                                   (1, 1712, 7360),     # 6.5 / 8.0
                                   (46, 1176, 8896),    # 9.0 / 9.3
                                   (16, 1424, 9600)],   # 9.5 / 9.9
                         ids=str)
def test_few_rows_wait_for_memory_with_four_lines(shape):
    for workspace in (True, False):
        ran = first_launch(*shape, workspace=workspace)
        assert ran.startswith("few_rows_bf16_16 ") and ran.endswith(" deep=1"), ran


# Rows of A (and of W) off lines, us: (not these): 256 x 256 tiles (dealt=1 or 2), ranges of steps (256 x 256: dealt=0)
@pytest.mark.parametrize("shape,pads,slower", [((658, 8696, 4736), (8, 0), "pg_bf16_t256"),     # 72 to 83 / 96
                                               ((3267, 2304, 2624), (8, 8), "pg_bf16_t256"),    # 43 / 56
                                               ((1190, 5416, 8064), (24, 0), "pg_bf16_t256"),   # 126 / 157
                                               ((514, 10120, 14720), (8, 0), "pg_bf16_t256"),   # 241 / 300
                                               ((714, 9888, 13056), (8, 0), "pg_bf16_t256"),    # 226 / 268
                                               ((1169, 5728, 15808), (24, 0), "pg_bf16_t256")], # 256 / 315
                         ids=str)
def test_rows_off_lines(shape, pads, slower):
    assert not first_launch(*shape, *pads).startswith(slower)


def test_ranges_are_dearer_off_lines_too():
    ran = first_launch(5506, 3616, 15744, 8, 8)   # 744 us in turn, 1026 in ranges
    assert ran.startswith("pg_bf16_t256_bf16 ") and ran[-1] in "12", ran
    ran = first_launch(318, 11384, 11840, 8)      # 180 us twice to a CU, 196 in ranges
    assert ran.startswith("pg_bf16_t128_bf16 ") and ran.endswith(" dealt=4"), ran


# Many rounds of tiles, rows on lines, us: as now / 128 x 128 tiles of two groups of waves
@pytest.mark.parametrize("shape,pad", [((2650, 12616, 9024), 64),    # 558 / 651
                                       ((2569, 6544, 1152), 0),      # 59 / 73
                                       ((548, 11520, 7808), 0)],     # 119 / 141
                         ids=str)
def test_many_rounds(shape, pad):
    ran = first_launch(*shape, pad)
    assert not (ran.startswith("pg_bf16_t128_bf16 ") and ran.endswith(" dealt=0")), ran
