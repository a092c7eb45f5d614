"""The plain product of lcma_gemm and lcma_gemm_nt on few tiles (csrc/lcma_small_plain.hip): every form, K that ends inside a line (what lies
behind a row of A, B or W is NaN and must not be read as part of it), rows and columns past the end of C, one line to many, both
layouts of B with the same bits.  Integer inputs are exact in any order of the sums; float inputs against 64 bits within the rounding of
C and of fp32 sums."""
import ctypes

import numpy as np
import pytest

import host_dispatch as D
import lcma_inputs as inp

gpu = pytest.mark.gpu

SHAPES = {"16": {(17, 40, 8): "t32x32x64_k4", (200, 200, 72): "t32x32x64_k4", (193, 1000, 328): "t32x32x64_k4", (400, 1000, 2056): "t32x32x64_k4",
                 (700, 704, 4104): "t64x64x64_k4", (1000, 520, 2040): "t64x64x64_k4", (1000, 1208, 1672): "t64x128x64_k2", (1100, 1000, 8200): "t64x128x64_k2",
                 (2284, 944, 4616): "t128x128x64_k2"},
          "f32": {(192, 200, 1992): "t32x32x32_k4", (193, 1000, 328): "t32x32x32_k4", (250, 252, 4100): "t32x32x32_k4", (1000, 516, 2040): "t32x32x32_k4"}}
CASES = [(dt, s) for dt in ("bf16", "f16", "f32") for s in SHAPES["f32" if dt == "f32" else "16"]]


@pytest.mark.parametrize("dt", ["bf16", "f16", "f32"])
def test_shapes_reach_their_kernels(dt):
    vec = 4 if dt == "f32" else 8
    for shape, name in SHAPES["f32" if dt == "f32" else "16"].items():
        for nk in (False, True):
            assert D.gemm(*shape, dt, None, nk, vec) == (0, [f"plain_{dt}_{name}" + "t" * nk]), shape
    # scaling, and what was chosen by name, stay where they were
    M, N, K = 400, 1000, 2056
    ran = D.call("lcma_gemm_ex", ctypes.c_float(2.0), ctypes.c_float(0.0), ctypes.c_int(0), M, N, K, D.A, K, D.B, N, D.C, N, ctypes.c_int(D.DTYPES[dt]),
                 ctypes.c_void_p(None), ctypes.c_void_p(None))
    assert ran[0] == 0 and "_c1" in ran[1][0], ran


@gpu
@pytest.mark.parametrize("dt,shape", CASES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v)
def test_both_layouts(dt, shape):
    import torch
    import gpu_util as G
    from paper_2605_06057_amd import binding as B
    M, N, K = shape
    td, vec = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}[dt], 4 if dt == "f32" else 8
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N + K)
    for kind in ("integers", "floats"):
        draw = (lambda r, c: torch.randint(-2, 3, (r, c), device="cuda", generator=gen).float()) if kind == "integers" else (lambda r, c: torch.randn((r, c), device="cuda", generator=gen))
        a, b, w = (torch.full((r, c + vec), float("nan"), device="cuda", dtype=td)[:, :c] for r, c in ((M, K), (K, N), (N, K)))
        a.copy_(draw(M, K))
        b.copy_(draw(K, N))
        w.copy_(b.t())
        got = []
        for name, call, right in (("lcma_gemm", B.lcma_gemm, b), ("lcma_gemm_nt", B.lcma_gemm_nt, w)):
            c = G.empty_like_c(M + 3, N + vec, dt, fill=float("nan"))
            print(f"small plain {name} {dt} {M}x{N}x{K} {kind}", flush=True)
            call(a, right, c[:M, :N])
            torch.cuda.synchronize()
            assert torch.isnan(c[M:]).all().item() and torch.isnan(c[:, N:]).all().item(), "wrote outside C"
            got.append(c[:M, :N])
        assert torch.equal(got[0], got[1])
        ref = a.double() @ b.double()
        if kind == "integers":
            assert torch.equal(got[0], ref.to(td))
        else:  # half an ulp of C (2^-8, 2^-11), or fp32 sums: 1e-6 covers 13 bits of random-walk growth of 2^-24
            assert ((got[0].double() - ref).norm() / ref.norm()).item() <= {"bf16": 2.0 ** -8, "f16": 2.0 ** -11, "f32": 1e-6}[dt]
