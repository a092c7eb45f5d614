"""The 128 x 128 and 64 x 128 tiles on which two groups of waves take the steps of K in turn (csrc/lcma_kpair.hpp): one to three steps, odd
numbers of them, more than a block of FP8 scale bytes, rows and columns past the end of C, K in slices, planes of Algorithm 1.  Integer
inputs (FP8: with another power of two for every 128 of a row) are exact in any order of the sums."""
import ctypes

import numpy as np
import pytest

import host_dispatch as D
import lcma_inputs as inp

gpu = pytest.mark.gpu

# shape: the launch by the library's rule with the workspace; dealt=0: 128 x 128, 3: slices, 4: the small tile twice to a CU, 5: 64 x 128
PLAIN = {(2050, 1096, 128): "t128_{0} jobs=153 units=153 ny=2 tail=128 panel=8 dealt=0", (1610, 2056, 1600): "t128_{0} jobs=221 units=221 ny=25 tail=128 panel=8 dealt=0",
         (743, 1400, 7168): "t128_{0} jobs=66 units=396 ny=112 tail=128 panel=8 dealt=3", (1300, 1400, 7104): "t128_{0} jobs=121 units=484 ny=111 tail=128 panel=8 dealt=3",
         (1025, 1400, 1088): "t128_{0} jobs=187 units=187 ny=17 tail=128 panel=8 dealt=5"}
FORCED = [(100, 72, 64), (300, 264, 192), (129, 136, 320), (300, 264, 448)]   # whole tiles in turn, which on 128 x 128 is this kernel
FP8 = {(613, 1000, 1600): 13, (930, 1688, 2184): 18, (1300, 2056, 3400): 27}


@pytest.mark.parametrize("dt", ["bf16", "f16"])
def test_shapes_reach_their_kernels(dt):
    whole = D.lib().lcma_split_group_scratch_bytes()
    for shape, want in PLAIN.items():
        ran = D.gemm_nt_ws(*shape, dt, whole)[1]
        assert ran[0] == f"pg_{dt}_" + want.format(dt), (shape, ran)
        assert (len(ran) == 2 and ran[1].startswith(f"few_rows_sum_{dt} ")) == ("dealt=3" in want), ran
    ran = D.gemm_nt_ws(500, 4096, 1024, dt, whole)[1]
    assert ran[0].startswith(f"few_rows_{dt}_64 ") and ran[0].endswith("deep=1"), ran
    for (M, N, K), steps in FP8.items():
        status, ran = D.call("lcma_fp8_gemm_nt", M, N, K, D.A, D.WORK, D.B, D.WORK + (1 << 36), D.C, N, ctypes.c_void_p(None))
        assert status == 0 and ran[0].startswith("pg_fp8_t128_bf16 ") and f" ny={steps} " in ran[0] and ran[0][-1] in "05", ran


@gpu
@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("shape", list(PLAIN) + [(500, 4096, 1024)] + FORCED, ids=lambda s: "x".join(map(str, s)))
def test_plain(dt, shape):
    import torch
    import gpu_util as G
    from paper_2605_06057_amd import binding as B
    M, N, K = shape
    Ai, Wi = inp.integers(61, 1, (M, K), -2, 2), inp.integers(61, 2, (N, K), -2, 2)
    a, w = (G.to_device(inp.store(x, dt), dt) for x in (Ai, Wi))
    want = inp.store(Ai.astype(np.float64) @ Wi.T.astype(np.float64), dt)
    ws = torch.full((B.lcma_split_group_scratch_bytes(),), 255, dtype=torch.uint8, device="cuda")  # NaN wherever it is read unwritten
    c = G.empty_like_c(M + 3, N + 8, dt, fill=float("nan"))
    print(f"kpair {dt} {M}x{N}x{K}", flush=True)
    B.lcma_set_tuning("schedule", "persist" if shape in FORCED else "")
    try:
        B.lcma_gemm_nt_ws(a, w, c[:M, :N], ws)
    finally:
        B.lcma_set_tuning("schedule", "")
    torch.cuda.synchronize()
    assert np.array_equal(G.to_host_stored(c[:M, :N], dt).view(np.uint8), want.view(np.uint8))
    assert torch.isnan(c[M:]).all().item() and torch.isnan(c[:, N:]).all().item(), "wrote outside C"


@gpu
@pytest.mark.parametrize("shape", list(FP8) + FORCED, ids=lambda s: "x".join(map(str, s)))
def test_fp8(shape):
    import torch
    from paper_2605_06057_amd import binding as B
    M, N, K = shape
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N + K)

    def operand(rows):  # integers of at most 2, 2^-2 to 2^2 times; a scale is exact for them
        x = torch.randint(-2, 3, (rows, K), device="cuda", generator=gen).double()
        e = torch.randint(-2, 3, (rows, -(-K // 128)), device="cuda", generator=gen)
        return x * torch.exp2(e.double()).repeat_interleave(128, dim=1)[:, :K]
    a, w = operand(M), operand(N)
    (aq, sa), (wq, sw) = B.lcma_fp8_quantize(a.bfloat16()), B.lcma_fp8_quantize(w.bfloat16())
    c = torch.full((M + 3, N + 8), float("nan"), dtype=torch.bfloat16, device="cuda")
    print(f"kpair fp8 {M}x{N}x{K}", flush=True)
    B.lcma_set_tuning("schedule", "persist" if shape in FORCED else "")
    try:
        B.lcma_fp8_gemm_nt(aq, sa, wq, sw, c[:M, :N], K)
    finally:
        B.lcma_set_tuning("schedule", "")
    torch.cuda.synchronize()
    assert torch.equal(c[:M, :N], (a @ w.t()).bfloat16())   # (sums below 2^24 sixteenths: exact in fp32)
    assert torch.isnan(c[M:]).all().item() and torch.isnan(c[:, N:]).all().item(), "wrote outside C"
