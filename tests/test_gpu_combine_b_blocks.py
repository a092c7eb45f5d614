"""Combine B of a K x N matrix, bit for bit against the oracle's, on both forms of the kernel (csrc/lcma_prepare_b.hpp): all blocks transposed
and the sums formed behind it (up to nine blocks), the sums first (sixteen).  Two tiles and a half along K/k, whole tiles along
N/n, every element of B another value, NaN around it."""
import numpy as np
import pytest

import lcma_inputs as inp
import oracle
from oracle import schemes as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("scheme", ["strassen", "laderman", "strassen2"])
def test_combine_b(scheme, dt):
    import torch
    import gpu_util as G
    from paper_2605_06057_amd import binding as B
    s = getattr(S, scheme)()
    N, K = s.n * 192, s.k * 160
    print(f"combine B {scheme} {dt} N={N} K={K}", flush=True)
    _, Bs = inp.matrices("uniform", "uniform", 8, N, K, dt, seed=41)
    wide = torch.full((K + 2, N + 16), float("nan"), dtype=G.empty_like_c(1, 1, dt).dtype, device="cuda")
    wide[1:K + 1, 8:N + 8] = G.to_device(Bs, dt)
    bt = B.lcma_prepare_b(wide[1:K + 1, 8:N + 8], B.lcma_scheme_load("builtin:" + scheme))
    got = bt.cpu().numpy().astype(np.float64).transpose(0, 2, 1)
    assert np.array_equal(got, oracle.combine_b_stored(s, inp.widen(Bs, dt), dt))
