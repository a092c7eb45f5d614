"""The 32 x 64 and 16 x 64 direct kernels for 16-bit products (csrc/lcma_direct16.hpp) at the edges of their pipelines: one step of 64 k to
a few more than stages, odd and even counts (two wave groups half a step or a step apart), a K that ends inside a step, edges of
the tile, rows of A and W that are a slice of a wider matrix; both layouts of B give the same bits."""
import pytest

import host_dispatch as D
import lcma_inputs as inp
import oracle

SHAPES = [(1, 8, 8), (63, 120, 128), (65, 136, 136), (64, 128, 256), (66, 264, 392), (33, 72, 520), (129, 200, 640), (40, 72, 840), (130, 136, 1096)]
LARGER_TILE = [(1000, 1544, 2056), (900, 2000, 2056), (2048, 1024, 1160)]   # more than a round of 16 x 64 tiles


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("shape", LARGER_TILE, ids=lambda s: "x".join(map(str, s)))
def test_more_than_a_round_of_small_tiles_takes_the_larger(shape, dtype):
    for nk in (False, True):
        assert D.gemm(*shape, dtype, "strassen", nk) == (0, [f"strassen_{dtype}_d32x64k4" + "t" * nk])


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("shape", SHAPES + LARGER_TILE[:1], ids=lambda s: "x".join(map(str, s)))
def test_tiles_layouts_and_slices(shape, dtype):
    import torch
    import gpu_util as G
    from paper_2605_06057_amd import binding as B
    M, N, K = shape
    As, Bs = inp.matrices("uniform", "uniform", M, N, K, dtype, 37)
    a, b = G.to_device(As, dtype), G.to_device(Bs, dtype)
    wide_a, wide_w = (torch.full((rows, K + 24), float("nan"), device="cuda", dtype=a.dtype) for rows in (M, N))   # NaN behind every row
    wide_a[:, :K] = a
    wide_w[:, :K] = b.t()
    ref = oracle.gemm(inp.widen(As, dtype), inp.widen(Bs, dtype))
    for name in (f"strassen_{dtype}_d32x64k4", f"strassen_{dtype}_d16x64k4"):
        c, ct, cs = (G.empty_like_c(M, N, dtype, fill=float("nan")) for _ in range(3))
        print(f"{name} {M}x{N}x{K}", flush=True)
        B.lcma_gemm_variant(name, a, b, c)
        B.lcma_gemm_variant(name + "t", a, b.t().contiguous(), ct, True)
        B.lcma_gemm_variant(name + "t", wide_a[:, :K], wide_w[:, :K], cs, True)
        torch.cuda.synchronize()
        assert oracle.rel_frobenius(G.to_host_f64(c, dtype), ref) <= 2e-2   # the bound of the 16-bit products
        assert torch.equal(c, ct) and torch.equal(c, cs)
