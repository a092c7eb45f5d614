"""The direct kernels for 16-bit products with few tiles (csrc/lcma_direct16.hpp): the same bits for both layouts of B, at one
element, a step that ends inside a lane's 32 bytes of K, fewer steps than waves, one more than a round of waves, edges of the
16 x 64 tile, and where lcma_gemm chooses them (CHOSEN); alpha and beta applied once, at every shape and with the 32 x 64 tile too.  (Exactness on integers, ragged edges and guard
rows: every variant, tests/test_gpu_parity.py.)"""
import pytest

import lcma_inputs as inp
import oracle

pytestmark = pytest.mark.gpu


CHOSEN = [(40, 72, 840), (64, 264, 840), (239, 376, 2056), (130, 1000, 1480)]   # by the library's rule, both types and layouts: test_dispatch.py


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("shape", [(1, 8, 8), (33, 136, 72), (64, 264, 520), (130, 1000, 648)] + CHOSEN, ids=lambda s: "x".join(map(str, s)))
def test_layouts_and_scaling(shape, dtype):
    import torch
    import gpu_util as G
    from paper_2605_06057_amd import binding as B
    M, N, K = shape
    s = B.lcma_scheme_load("builtin:strassen")
    As, Bs = inp.matrices("uniform", "uniform", M, N, K, dtype, 23)
    a, b = G.to_device(As, dtype), G.to_device(Bs, dtype)
    w = b.t().contiguous()
    c, ct, d, e = (G.empty_like_c(M, N, dtype, fill=float("nan")) for _ in range(4))
    name = f"strassen_{dtype}_d16x64k4"
    print(f"{name} {M}x{N}x{K}", flush=True)
    B.lcma_gemm_variant(name, a, b, c)
    B.lcma_gemm_variant(name + "t", a, w, ct, True)
    B.lcma_gemm(a, b, d, s)
    B.lcma_gemm_nt(a, w, e, s)
    torch.cuda.synchronize()
    ref = oracle.gemm(inp.widen(As, dtype), inp.widen(Bs, dtype))
    assert oracle.rel_frobenius(G.to_host_f64(c, dtype), ref) <= 2e-2   # the bound of the 16-bit products
    assert torch.equal(c, ct) and torch.equal(d, e)
    if shape in CHOSEN:
        assert torch.equal(c, d)
    old = (torch.arange(M * N, device="cuda", dtype=torch.float32).view(M, N) / (M * N)).to(c.dtype)
    for tile in (16, 32):
        name = f"strassen_{dtype}_d{tile}x64k4"
        print(f"{name} {M}x{N}x{K} alpha, beta", flush=True)
        B.lcma_gemm_variant(name, a, b, c)
        y, z = old.clone(), old.clone()
        for right, out, variant, nk in ((b, y, name, False), (w, z, name + "t", True)):
            B.lcma_set_tuning("variant", variant)
            try:
                B.lcma_gemm_ex(0.5, -2.0, a, right, out, s, b_nk=nk)
            finally:
                B.lcma_set_tuning("variant", "")
        torch.cuda.synchronize()
        assert torch.equal(y, z)
        # c rounded once (half an ulp of c, u = 2^-9 or 2^-12 of its magnitude, halved by alpha), then the sum rounded once
        u = 2.0 ** (-9 if dtype == "bf16" else -12)
        want = 0.5 * c.double() - 2.0 * old.double()
        assert ((y.double() - want).abs() <= 2 * u * (c.double().abs() + want.abs()) + 1e-7).all().item()


# K of a step and less, of a step that ends inside a lane's 32 bytes, and more steps than waves
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("shape", [(17, 72, 64), (33, 136, 72), (50, 200, 1096)], ids=lambda s: "x".join(map(str, s)))
def test_weights_whose_rows_start_on_lines(shape, dtype):
    import torch
    import gpu_util as G
    from paper_2605_06057_amd import binding as B
    M, N, K = shape
    As, Bs = inp.matrices("uniform", "uniform", M, N, K, dtype, 29)
    a, b = G.to_device(As, dtype), G.to_device(Bs, dtype)
    wide = torch.full((N, (K + 63) // 64 * 64), float("nan"), device="cuda", dtype=b.dtype)   # NaN behind every row
    wide[:, :K] = b.t()
    c, ct = (G.empty_like_c(M, N, dtype, fill=float("nan")) for _ in range(2))
    name = f"strassen_{dtype}_d16x64k4"
    print(f"{name}t {M}x{N}x{K} row pitch {wide.stride(0)}", flush=True)
    B.lcma_gemm_variant(name, a, b, c)
    B.lcma_gemm_variant(name + "t", a, wide[:, :K], ct, True)
    torch.cuda.synchronize()
    ref = oracle.gemm(inp.widen(As, dtype), inp.widen(Bs, dtype))
    assert oracle.rel_frobenius(G.to_host_f64(c, dtype), ref) <= 2e-2   # the bound of the 16-bit products
    assert torch.equal(c, ct)


# measured: 13.4 and 12.9 us against 18.0 and 14.8; 14.1 and 13.4 against 18.2 and 15.0; 20.5 and 18.9 against 29.3 and 23.0
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("shape", [(101, 456, 1024), (312, 520, 1024), (63, 312, 2048)], ids=lambda s: "x".join(map(str, s)))
def test_neither_layout_is_slower_than_the_staged_kernel(shape, dtype):
    """Both layouts of B make one choice (they give the same bits), so the direct kernel has to be the faster one for both; weights
    whose rows are whole lines are its slowest operand."""
    import torch
    import gpu_util as G
    from paper_2605_06057_amd import binding as B
    M, N, K = shape
    As, Bs = inp.matrices("uniform", "uniform", M, N, K, dtype, 31)
    a, b = G.to_device(As, dtype), G.to_device(Bs, dtype)
    w, c = b.t().contiguous(), G.empty_like_c(M, N, dtype)

    def graph(fn):
        fn()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            for _ in range(20):
                fn()
        g.replay()
        return g

    for right, nk, names in ((b, False, ("t64x64x32_c7fio2", "d16x64k4")), (w, True, ("t64x64x32_c7fito2", "d16x64k4t"))):
        graphs = [graph(lambda: B.lcma_gemm_variant(f"strassen_{dtype}_{v}", a, right, c, nk)) for v in names]
        best = [float("inf")] * 2
        for _ in range(7):
            for i, g in enumerate(graphs):
                e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                e0.record()
                g.replay()
                e1.record()
                torch.cuda.synchronize()
                best[i] = min(best[i], e0.elapsed_time(e1) / 20 * 1e3)
        print(f"{dtype} {M}x{N}x{K}{' N x K' if nk else ''}: staged {best[0]:.1f} us, direct {best[1]:.1f}", flush=True)
        assert best[1] <= 1.05 * best[0], (nk, best)
