"""Algorithm 1 in 16 bit with blocks of rows cut at whole 16 rows (csrc/unfused.cc): every kernel of the batched stage with tiles that hang over
the end of a plane, a last block that is short or empty, the planes of static weights kept while M and with it the cut changes.  Integer
inputs are exact."""
import ctypes

import numpy as np
import pytest

import host_dispatch as D
import lcma_inputs as inp
import oracle

gpu = pytest.mark.gpu

# the first M is cut at 16 rows (144 instead of 256; 272 / 384), the second at whole tiles; <3,3,3;23> is left at whole tiles by both
CASES = [("strassen2", "bf16", (545, 500, 1464, 1288)), ("laderman", "f16", (577, 700, 1600, 1160)), ("strassen", "bf16", (523, 508, 3976, 2312))]


# rows of a block, tile and how the tile-products are dealt (0: a work-group each, 1: 256 x 256 in turn, 4: 128 x 128 twice to a CU, 5: 64 x 128,
# "split": ranges of steps) and rows of the last block
KERNELS = [("strassen2", "bf16", (518, 536, 1824), 144, "t128_f16", "0", 86), ("laderman", "f16", (213, 2232, 2176), 80, "t128_f32", "0", 53),
           ("strassen2", "bf16", (24, 632, 304), 16, "t128_f16", "4", 0), ("laderman", "f16", (23, 816, 376), 16, "t128_f32", "4", 0),
           ("strassen2", "bf16", (52, 304, 1128), 16, "t128_f16", "5", 4), ("laderman", "f16", (22, 392, 664), 16, "t128_f32", "5", 0),
           ("strassen2", "bf16", (514, 2800, 336), 144, "t256_f16", "0", 82), ("laderman", "f16", (786, 2640, 336), 272, "t256_f32", "0", 242),
           ("strassen2", "bf16", (532, 3152, 3048), 144, "t256_f16", "1", 100),
           ("strassen2", "bf16", (518, 536, 1824), 144, "t128_f16", "split", 86), ("laderman", "f16", (213, 2232, 2176), 80, "t128_f32", "split", 53)]


@pytest.mark.parametrize("name,dt,shape,rows,tile,dealt,last", KERNELS, ids=str)
def test_the_cut_and_the_kernel(name, dt, shape, rows, tile, dealt, last):
    L, s = D.lib(), D.Scheme(name)
    M, N, K = shape
    f = L.lcma_unfused_workspace_bytes
    f.restype = ctypes.c_int64
    need = f(*(ctypes.c_int64(x) for x in shape), ctypes.c_int(D.DTYPES[dt]), s.handle)
    L.lcma_set_tuning(b"schedule", b"split" if dealt == "split" else b"")
    try:
        status, ran = D.call("lcma_gemm_unfused", ctypes.c_int(1), M, N, K, D.A, K, D.B, N, D.C, N, ctypes.c_int(D.DTYPES[dt]), s, D.WORK,
                             need + L.lcma_split_group_scratch_bytes(), ctypes.c_int(0), ctypes.c_void_p(None))
    finally:
        L.lcma_set_tuning(b"schedule", b"")
    stage = [x for x in ran if x.startswith("pg_")]
    assert status == 0 and len(stage) == 1 and stage[0].startswith(f"pg_f16_{tile} "), ran
    jobs, units = (int(stage[0].split(k + "=")[1].split()[0]) for k in ("jobs", "units"))
    assert stage[0].endswith(" dealt=" + ("0" if dealt == "split" else dealt)) and (units == jobs or dealt != "0"), stage
    assert dealt != "split" or units > jobs, stage
    blocks = {"strassen2": 4, "laderman": 3}[name]
    assert L.dispatch_plane_rows() == rows and max(0, M - (blocks - 1) * rows) == last


@gpu
@pytest.mark.parametrize("name,dt,shape,rows,tile,dealt,last", KERNELS, ids=str)
def test_every_kernel_on_cut_planes(name, dt, shape, rows, tile, dealt, last):
    import torch
    import gpu_util as G
    from paper_2605_06057_amd import binding as B
    M, N, K = shape
    h = B.lcma_scheme_load("builtin:" + name)
    nbytes = B.lcma_unfused_workspace_bytes(h, M, N, K, B.DTYPE_IDS[dt]) + B.lcma_split_group_scratch_bytes()
    ws = torch.full((nbytes,), 0x7f, dtype=torch.uint8, device="cuda")   # stale bytes: what is read is written before
    Ai, Bi = inp.integers(53, M, (M, K), -1, 1), inp.integers(53, 2, (K, N), -1, 1)
    want = inp.store(oracle.gemm(Ai, Bi).astype(np.float64), dt)
    c = G.empty_like_c(M + 3, N + 8, dt, fill=float("nan"))
    print(f"cut planes {name} {dt} {M}x{N}x{K} {tile} dealt {dealt}", flush=True)
    B.lcma_set_tuning("schedule", "split" if dealt == "split" else "")
    try:
        B.lcma_gemm_unfused(1, G.to_device(inp.store(Ai, dt), dt), G.to_device(inp.store(Bi, dt), dt), c[:M, :N], h, ws)
    finally:
        B.lcma_set_tuning("schedule", "")
    torch.cuda.synchronize()
    assert np.array_equal(G.to_host_stored(c[:M, :N], dt).view(np.uint8), want.view(np.uint8))
    assert torch.isnan(c[M:]).all().item() and torch.isnan(c[:, N:]).all().item(), "wrote outside C"


@gpu
@pytest.mark.parametrize("name,dt,shape", CASES, ids=lambda c: str(c))
def test_cut_at_sixteen_rows(name, dt, shape):
    import torch
    import gpu_util as G
    from paper_2605_06057_amd import binding as B
    M1, M2, N, K = shape
    h = B.lcma_scheme_load("builtin:" + name)
    nbytes = max(B.lcma_unfused_workspace_bytes(h, M, N, K, B.DTYPE_IDS[dt]) for M in (M1, M2))
    ws = torch.full((nbytes,), 0x7f, dtype=torch.uint8, device="cuda")   # stale bytes: what is read is written before
    Bi = inp.integers(52, 2, (K, N), -1, 1)
    b = G.to_device(inp.store(Bi, dt), dt)
    for M, reuse in ((M1, False), (M2, True), (M1, True)):
        Ai = inp.integers(51, M, (M, K), -1, 1)
        want = inp.store(oracle.gemm(Ai, Bi).astype(np.float64), dt)
        c = G.empty_like_c(M + 3, N + 8, dt, fill=float("nan"))
        print(f"row blocks {name} {dt} {M}x{N}x{K} reuse {reuse}", flush=True)
        B.lcma_gemm_unfused(1, G.to_device(inp.store(Ai, dt), dt), b, c[:M, :N], h, ws, reuse_bt=reuse)
        torch.cuda.synchronize()
        assert np.array_equal(G.to_host_stored(c[:M, :N], dt).view(np.uint8), want.view(np.uint8))
        assert torch.isnan(c[M:]).all().item() and torch.isnan(c[:, N:]).all().item(), "wrote outside C"
