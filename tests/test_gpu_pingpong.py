"""The 256 x 256 plane GEMM with the two waves of a SIMD in turn (csrc/lcma_pingpong.hpp), forced through the "persist"
schedule, at the sizes where its pipeline can go wrong: one, two and three steps of K (an odd number is rounded up by a step of
zeros), tile-products that follow each other in a work-group (306 tiles on 256 work-groups, dealt both ways), groups of
four scale bytes that end inside a tile-product, tiles that hang over the end of a plane, ragged edges.  Integer inputs:
every product and sum is exact, so the oracle's bits are the only right answer."""
import numpy as np
import pytest

import lcma_inputs as inp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2605_06057_amd import binding
    binding.lib()
    binding.lcma_set_tuning("schedule", "persist")
    yield binding
    binding.lcma_set_tuning("schedule", "")


def _check(c, M, N, want, dt):
    import torch
    import gpu_util as G
    torch.cuda.synchronize()
    assert np.array_equal(G.to_host_stored(c[:M, :N], dt).view(np.uint8), want.view(np.uint8))
    assert torch.isnan(c[M:]).all().item() and torch.isnan(c[:, N:]).all().item(), "wrote outside C"


@pytest.mark.parametrize("shape", [(8, 8, 64), (257, 264, 128), (500, 1032, 192), (4352, 4608, 64), (4352, 4608, 192), (4200, 4608, 256)],
                         ids=lambda s: "x".join(map(str, s)))
def test_plain(B, shape):
    import torch
    import gpu_util as G
    M, N, K = shape
    Ai, Wi = inp.integers(91, 1, (M, K)), inp.integers(91, 2, (N, K))
    c = G.empty_like_c(M + 3, N + 8, "bf16", fill=float("nan"))
    print(f"ping-pong bf16 {M}x{N}x{K}", flush=True)
    B.lcma_gemm_nt_ws(G.to_device(inp.store(Ai, "bf16"), "bf16"), G.to_device(inp.store(Wi, "bf16"), "bf16"), c[:M, :N], None)
    _check(c, M, N, inp.store(Ai.astype(np.float64) @ Wi.T.astype(np.float64), "bf16"), "bf16")


@pytest.mark.parametrize("shape", [(8, 8, 128), (300, 264, 384), (4352, 4608, 384), (4352, 4608, 640)], ids=lambda s: "x".join(map(str, s)))
def test_fp8(B, shape):
    import torch
    import gpu_util as G
    M, N, K = shape
    Ai, Wi = inp.integers(92, 1, (M, K)), inp.integers(92, 2, (N, K))
    dev = lambda x: G.to_device(inp.store(x, "bf16"), "bf16")
    ops = []
    for x in (Ai, Wi):  # the scale bytes behind the last block of a row are nobody's: as NaN they must not matter
        S = torch.full((x.shape[0], -(-K // 512) * 4), 255, dtype=torch.uint8, device="cuda")
        ops += list(B.lcma_fp8_quantize(dev(x), None, S))
    c = G.empty_like_c(M + 3, N + 8, "bf16", fill=float("nan"))
    print(f"ping-pong fp8 {M}x{N}x{K}", flush=True)
    B.lcma_fp8_gemm_nt(*ops, c[:M, :N], K)
    _check(c, M, N, inp.store(Ai.astype(np.float64) @ Wi.T.astype(np.float64), "bf16"), "bf16")


# planes of 384 and 640 rows or columns (multiples of 128 only); fp16 and fp32 products; 7 x 6 x 9 = 378 tile-products
@pytest.mark.parametrize("dt,name,shape", [("bf16", "strassen", (700, 1200, 136)), ("f16", "strassen", (700, 1200, 136)),
                                           ("bf16", "strassen", (2600, 4400, 328)), ("f16", "laderman", (1100, 1160, 200))])
def test_planes_that_are_no_whole_tiles(B, dt, name, shape):
    import torch
    import gpu_util as G
    M, N, K = shape
    h = B.lcma_scheme_load("builtin:" + name)
    Ai, Bi = inp.integers(93, 1, (M, K), -1, 1), inp.integers(93, 2, (K, N), -1, 1)
    ws = torch.empty((B.lcma_unfused_workspace_bytes(h, M, N, K, B.DTYPE_IDS[dt]),), dtype=torch.uint8, device="cuda")
    c = G.empty_like_c(M + 3, N + 8, dt, fill=float("nan"))
    print(f"ping-pong planes {dt} {name} {M}x{N}x{K}", flush=True)
    B.lcma_gemm_unfused(1, G.to_device(inp.store(Ai, dt), dt), G.to_device(inp.store(Bi, dt), dt), c[:M, :N], h, ws)
    _check(c, M, N, inp.store(Ai.astype(np.float64) @ Bi.astype(np.float64), dt), dt)
