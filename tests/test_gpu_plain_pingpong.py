"""The plain 16-bit product on the ping-pong kernels (csrc/lcma_pingpong.hpp, lcma_pingpong_narrow.hpp) where lcma_gemm, lcma_gemm_nt
and lcma_gemm_nt_ws choose them: K that ends inside a step of 64 (what lies behind a row of A or W is NaN and must not be
read as part of it), ragged M and N, both tiles and both layouts of B.  lcma_gemm's results are those of
the generated kernels bit for bit, which is what the float inputs are compared with."""
import numpy as np
import pytest

import lcma_inputs as inp

pytestmark = pytest.mark.gpu

# What the library takes for rows that start on lines (test_dispatch.py holds it to that, both types).  256 x 128 tiles: 8 to 65 steps of K,
# 8 elements or a whole step in the last, 32 to 660 tiles (256 work-groups run at a time)
NARROW = [(1000, 4104, 456), (520, 8200, 648), (1000, 4104, 960), (1000, 4104, 1032), (1000, 4104, 1096), (5000, 4104, 1032), (520, 8200, 4104),
          (2040, 2056, 4104)]
# 256 x 256: 10 to 65 steps, 56, 8 and 64 elements in the last; 132 tiles (dealt in rounds), 561 (two and three to a work-group, an
# eighth to every XCD), a long K
WIDE = [(1000, 8200, 632), (1000, 8200, 832), (1000, 8200, 840), (4100, 8200, 1144), (4100, 2056, 4104)]
# (N x K weights stay with the generated kernel here)
KN_ONLY = [(1000, 4104, 456), (520, 8200, 648)]
SHAPES = NARROW + WIDE


def pitch(n):
    """Row pitch: at least one unused column, rows on 128-byte lines."""
    return n // 64 * 64 + 64


@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_same_bits_as_the_generated_kernels(dt, shape):
    import torch
    import gpu_util as G
    from paper_2605_06057_amd import binding as B
    M, N, K = shape
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N + K)
    td = {"bf16": torch.bfloat16, "f16": torch.float16}[dt]
    nan = lambda r, c: torch.full((r, c), float("nan"), device="cuda", dtype=td)
    a, b, w = nan(M, pitch(K)), nan(K, pitch(N)), nan(N, pitch(K))
    a[:, :K] = torch.randn((M, K), device="cuda", generator=gen)
    b[:, :N] = torch.randn((K, N), device="cuda", generator=gen) * 0.05
    w[:, :K] = b[:, :N].t()
    a, b, w = a[:, :K], b[:, :N], w[:, :K]
    want = G.empty_like_c(M, N, dt, fill=float("nan"))
    B.lcma_gemm_variant(f"plain_{dt}_t128x128x64_c1o2", a, b, want)
    for name, call in (("lcma_gemm", lambda c: B.lcma_gemm(a, b, c)), ("lcma_gemm_nt", lambda c: B.lcma_gemm_nt(a, w, c)),
                       ("lcma_gemm_ex", lambda c: B.lcma_gemm_ex(1.0, 0.0, a, b, c)), ("lcma_gemm_ex N x K", lambda c: B.lcma_gemm_ex(1.0, 0.0, a, w, c, None, True))):
        c = G.empty_like_c(M + 3, N + 8, dt, fill=float("nan"))
        print(f"plain {name} {dt} {M}x{N}x{K}", flush=True)
        call(c[:M, :N])
        torch.cuda.synchronize()
        assert torch.equal(c[:M, :N], want), name
        assert torch.isnan(c[M:]).all().item() and torch.isnan(c[:, N:]).all().item(), "wrote outside C"
    rows = torch.arange(0, M, max(1, M // 37), device="cuda")
    ref = a[rows].double() @ b.double()
    err = (want[rows].double() - ref).norm() / ref.norm()
    assert err.item() <= 2.0 ** (-9 if dt == "bf16" else -12) + 1e-5   # the rounding of C and fp32 sums of K terms


@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("shape", [(2048, 4096, 1024), (1000, 3000, 4160)], ids=lambda s: "x".join(map(str, s)))
def test_exact_on_integers_with_a_workspace(dt, shape):
    import torch
    import gpu_util as G
    from paper_2605_06057_amd import binding as B
    M, N, K = shape
    Ai, Wi = inp.integers(95, 1, (M, K), -2, 2), inp.integers(95, 2, (N, K), -2, 2)
    c = G.empty_like_c(M + 3, N + 8, dt, fill=float("nan"))
    ws = torch.empty((B.lcma_split_group_scratch_bytes(),), dtype=torch.uint8, device="cuda")
    print(f"plain lcma_gemm_nt_ws {dt} {M}x{N}x{K}", flush=True)
    B.lcma_gemm_nt_ws(G.to_device(inp.store(Ai, dt), dt), G.to_device(inp.store(Wi, dt), dt), c[:M, :N], ws)
    torch.cuda.synchronize()
    want = inp.store(Ai.astype(np.float64) @ Wi.T.astype(np.float64), dt)
    assert np.array_equal(G.to_host_stored(c[:M, :N], dt).view(np.uint8), want.view(np.uint8))
    assert torch.isnan(c[M:]).all().item() and torch.isnan(c[:, N:]).all().item(), "wrote outside C"
