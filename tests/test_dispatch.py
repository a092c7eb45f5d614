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
