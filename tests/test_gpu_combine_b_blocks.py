"""Combine B of a K x N matrix, bit for bit against the oracle's, on both forms of the kernel (csrc/lcma_prepare_b.hpp): all blocks transposed
and the sums formed behind it (up to nine blocks), the sums first (sixteen).  A tile is 64 k (fp32: 32): two and a half of them along K/k
in 16 bit, five and a half in fp32, and blocks that the end of B cuts short along both; every element of B another value, NaN around it."""
import numpy as np
import pytest

import lcma_inputs as inp
import oracle
from oracle import schemes as S

pytestmark = pytest.mark.gpu


CASES = [(scheme, dt) for scheme in ("strassen", "laderman", "strassen2") for dt in ("bf16", "f16", "f32") if (scheme, dt) != ("strassen2", "f16")]


@pytest.mark.parametrize("bk,short", [(160, (0, 0)), (176, (0, 0)), (176, (24, 40))], ids=str)
@pytest.mark.parametrize("scheme,dt", CASES)
def test_combine_b(scheme, dt, bk, short):
    import torch
    import gpu_util as G
    from paper_2605_06057_amd import binding as B
    s = getattr(S, scheme)()
    N, K = s.n * 192 - short[1], s.k * bk - short[0]
    print(f"combine B {scheme} {dt} N={N} K={K}", flush=True)
    _, Bs = inp.matrices("uniform", "uniform", 8, N, K, dt, seed=41)
    wide = torch.full((K + 2, N + 16), float("nan"), dtype=G.empty_like_c(1, 1, dt).dtype, device="cuda")
    wide[1:K + 1, 8:N + 8] = G.to_device(Bs, dt)
    bt = B.lcma_prepare_b(wide[1:K + 1, 8:N + 8], B.lcma_scheme_load("builtin:" + scheme))
    padded = np.zeros((s.k * bt.shape[2], s.n * bt.shape[1]))   # the planes are cut from B with zeros up to whole granules
    padded[:K, :N] = inp.widen(Bs, dt)
    got = bt.cpu().numpy().astype(np.float64).transpose(0, 2, 1)
    assert np.array_equal(got, oracle.combine_b_stored(s, padded, dt))
