"""Algorithm 1 in 16 bit with blocks of rows cut at whole 16 rows (csrc/unfused.cc): tiles that hang over the end of a plane, a last block
that is short or empty, the planes of static weights kept while M and with it the cut changes.  Integer inputs are exact."""
import numpy as np
import pytest

import lcma_inputs as inp
import oracle

pytestmark = pytest.mark.gpu

# the first M is cut at 16 rows (144 instead of 256, 208 / 256, 272 / 384), the second at whole tiles
CASES = [("strassen2", "bf16", (545, 500, 1464, 1288)), ("laderman", "f16", (577, 700, 1600, 1160)), ("strassen", "bf16", (523, 508, 3976, 2312))]


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
