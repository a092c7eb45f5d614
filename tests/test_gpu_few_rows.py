"""lcma_gemm_nt_ws on few rows or a small C (csrc/lcma_few_rows.hpp): tiles of 16, 32 and 64, K in one piece and in slices (the
last one shorter), rows and columns past the end of C, with the workspace and without.  Integer inputs are exact in any order
of the sums; float inputs against the fp64 product within the rounding of C plus that of fp32 sums over K."""
import numpy as np
import pytest

import lcma_inputs as inp
import oracle

pytestmark = pytest.mark.gpu

# shape: (tile, slices of K) with the workspace and without it, by the library's rule (test_dispatch.py holds it to that)
PLANS = {(1, 8, 1024): ((16, 1), (16, 1)), (1, 1000, 2048): ((16, 1), (16, 1)), (17, 72, 192): ((16, 1), (16, 1)), (33, 1000, 576): ((16, 1), (16, 1)),
         (100, 520, 4160): ((16, 1), (16, 1)), (300, 520, 1024): ((32, 1), (32, 1)), (64, 4096, 4096): ((32, 1), (32, 1)),
         (65, 4088, 4160): ((64, 2), (32, 1)),      # 130 steps of 32 in slices of 72: the last one of 58
         (755, 96, 10368): ((64, 9), (16, 1)),      # 324 steps in slices of 40: the last one of 4
         (64, 4096, 14336): ((64, 4), (32, 1)), (65, 4088, 8256): ((64, 2), (64, 1)),
         (129, 200, 14400): ((16, 1), (16, 1)),     # eight waves with four lines in flight, the last turn of two waves only
         (250, 2000, 2112): ((32, 1), (32, 1)), (40, 14344, 1024): ((64, 1), (64, 1))}
SHAPES = list(PLANS)


@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_few_rows(dt, shape):
    import torch
    import gpu_util as G
    from paper_2605_06057_amd import binding as B
    M, N, K = shape
    Ai, Wi = inp.integers(81, 1, (M, K + 8), -2, 2), inp.integers(81, 2, (N, K), -2, 2)
    dev = lambda x: G.to_device(inp.store(x, dt), dt)
    ws = torch.full((B.lcma_split_group_scratch_bytes(),), 255, dtype=torch.uint8, device="cuda")  # NaN wherever it is read unwritten
    want = inp.store(Ai[:, :K].astype(np.float64) @ Wi.T.astype(np.float64), dt)
    a, w = dev(Ai)[:, :K], dev(Wi)
    for space in (ws, None):
        c = G.empty_like_c(M + 3, N + 8, dt, fill=float("nan"))
        print(f"few rows {dt} {M}x{N}x{K} workspace {space is not None}", flush=True)
        B.lcma_gemm_nt_ws(a, w, c[:M, :N], space)
        torch.cuda.synchronize()
        assert np.array_equal(G.to_host_stored(c[:M, :N], dt).view(np.uint8), want.view(np.uint8))
        assert torch.isnan(c[M:]).all().item() and torch.isnan(c[:, N:]).all().item(), "wrote outside C"
    rng = np.random.default_rng(M + N + K)
    Af, Wf = inp.store(rng.standard_normal((M, K)), dt), inp.store(rng.standard_normal((N, K)) * 0.05, dt)
    c = G.empty_like_c(M, N, dt, fill=float("nan"))
    B.lcma_gemm_nt_ws(G.to_device(Af, dt), G.to_device(Wf, dt), c, ws)
    ref = oracle.gemm(inp.widen(Af, dt), np.ascontiguousarray(inp.widen(Wf, dt).T))
    # fp32 sums of K terms, and the one rounding of C: on one value at most half an ulp, 2^-8 (2^-11) of it; over many the root mean
    # square, ulp / sqrt(12) against 1.5 in the middle of a binade, is 2^-9.4 (2^-12.4).  So half of it where there are many values.
    u = 2.0 ** (-8 if dt == "bf16" else -11)
    assert oracle.rel_frobenius(G.to_host_f64(c, dt), ref) <= (u if M * N < 1000 else u / 2) + 1e-5


# Many rows and few columns: fewer blocks of columns (and slices of K) than XCDs.  Measured, this kernel / the plane GEMM, us: 34 / 48 (97 on two XCDs), 7.2 / 7.4 (17.6)
@pytest.mark.parametrize("shape", [(4266, 128, 4288), (5369, 192, 512)], ids=lambda s: "x".join(map(str, s)))
def test_few_columns_are_no_slower_than_one_tile_per_work_group(shape):
    import torch
    from paper_2605_06057_amd import binding as B
    M, N, K = shape
    a, w = torch.randn((M, K), device="cuda").half(), torch.randn((N, K), device="cuda").half()
    c = torch.empty((M, N), device="cuda", dtype=torch.float16)
    ws = torch.empty((B.lcma_split_group_scratch_bytes(),), dtype=torch.uint8, device="cuda")
    graphs = []
    for schedule in ("static", ""):
        B.lcma_set_tuning("schedule", schedule)
        B.lcma_gemm_nt_ws(a, w, c, ws)
        torch.cuda.synchronize()
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1]):
            for _ in range(20):
                B.lcma_gemm_nt_ws(a, w, c, ws)
    best = [float("inf")] * 2
    for _ in range(7):
        for i, g in enumerate(graphs):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            g.replay()
            e1.record()
            torch.cuda.synchronize()
            best[i] = min(best[i], e0.elapsed_time(e1) / 20 * 1e3)
    print(f"{M}x{N}x{K}: static {best[0]:.1f} us, chosen {best[1]:.1f}", flush=True)
    assert best[1] <= 1.15 * best[0], best
