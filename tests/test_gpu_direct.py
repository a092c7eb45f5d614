"""The direct kernels for small fp32 products (csrc/lcma_direct.hpp) where lcma_gemm chooses them: the same bits for both
layouts of B and through lcma_gemm_ex with alpha = 1, beta = 0, alpha and beta applied once, one group of 16 elements of K for
eight waves, blocks with more padding than content.  (Exactness on integers, ragged edges and guard rows: every variant,
tests/test_gpu_parity.py.)"""
import numpy as np
import pytest

import lcma_inputs as inp
import oracle

pytestmark = pytest.mark.gpu


# tiles of 16, and of 32 (857 x 1048 x 808): test_dispatch.py; 3 x 4 x 4 stays with the staged kernel
SHAPES = [(3, 4, 4), (3, 4, 16), (33, 36, 20), (256, 256, 256), (130, 516, 1000), (700, 712, 404), (857, 1048, 808)]


@pytest.mark.parametrize("scheme", ["strassen", "winograd"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_layouts_and_scaling(scheme, shape):
    import torch
    import gpu_util as G
    from paper_2605_06057_amd import binding as B
    M, N, K = shape
    s = B.lcma_scheme_load("builtin:" + scheme)
    As, Bs = inp.matrices("uniform", "uniform", M, N, K, "f32", 17)
    a, b = G.to_device(As, "f32"), G.to_device(Bs, "f32")
    c, ct, cx = (G.empty_like_c(M, N, "f32", fill=float("nan")) for _ in range(3))
    print(f"direct {scheme} {M}x{N}x{K}", flush=True)
    B.lcma_gemm(a, b, c, s)
    B.lcma_gemm_nt(a, b.t().contiguous(), ct, s)
    B.lcma_gemm_ex(1.0, 0.0, a, b, cx, s)
    torch.cuda.synchronize()
    ref = oracle.gemm(inp.widen(As, "f32"), inp.widen(Bs, "f32"))
    assert oracle.rel_frobenius(G.to_host_f64(c, "f32"), ref) <= 1e-5
    assert torch.equal(c, ct) and torch.equal(c, cx)
    old = torch.arange(M * N, device="cuda", dtype=torch.float32).view(M, N) / (M * N)
    y = old.clone()
    B.lcma_gemm_ex(0.5, -2.0, a, b, y, s, b_nk=False)
    want = 0.5 * c.double() - 2.0 * old.double()   # from the unscaled fp32 result: alpha exact, one rounding of the sum
    assert ((y.double() - want).abs() <= 2.0 ** -24 * want.abs() + 1e-30).all().item()
