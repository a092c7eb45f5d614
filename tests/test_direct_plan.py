"""What the generator plans for the direct kernels (gen/generate.py), which its budgets are checked against, is what the kernels have."""
import os
import re
import shutil

import pytest

from paper_2605_06057_amd import build
from test_lds_reuse import compiled

# accumulator registers per lane: seven products, a wave's part of the tile over 64 lanes
KERNELS = {"strassen_bf16_d32x64k4": 7 * 32 * 32 // 64, "strassen_f16_d16x64k4t": 7 * 16 * 32 // 64, "strassen_bf16_d16x64k4": 7 * 16 * 32 // 64,
           "strassen_f32_d32x32k8": 7 * 32 * 32 // 64, "winograd_f32_d16x16k8t": 7 * 16 * 16 // 64}


@pytest.mark.skipif(not (os.path.exists(build.HIPCC) or shutil.which(build.HIPCC)), reason="needs hipcc")
@pytest.mark.parametrize("name", KERNELS)
def test_planned_registers_and_lds(name, tmp_path):
    from paper_2605_06057_amd.gen import generate as G
    schemes = G.load_schemes()
    variant = next(v for v in G.manifest(schemes) if v.name == name)
    regs, lds = G.plan(schemes[variant.scheme], variant)[:2]
    source = os.path.join(build.GEN, f"k_{name}.hip")
    if not os.path.exists(source):
        G.generate(build.GEN)
    held = int(re.search(r"E4smem = .*?\[(\d+) x i8\]", compiled(source, tmp_path)).group(1))
    assert (regs, lds) == (KERNELS[name], held)
