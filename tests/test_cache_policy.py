"""Cache policy of the loads of Combine H (csrc/lcma_combine_h.hpp): the planes of 16-bit results are read streamed, those of fp32 results with the
ordinary policy.  From the compiler's own output."""
import os
import re
import shutil

import pytest

from paper_2605_06057_amd import build
from test_lds_reuse import compiled, kernels


@pytest.mark.skipif(not (os.path.exists(build.HIPCC) or shutil.which(build.HIPCC)), reason="needs hipcc")
@pytest.mark.parametrize("dtype,planes,policies", [("f32", "h", {"0"}), ("f16", "h32", {"2"})])
def test_planes_of_combine_h(dtype, planes, policies, tmp_path):
    source = os.path.join(build.GEN, f"k_stage_strassen_{dtype}.hip")
    if not os.path.exists(source):
        from paper_2605_06057_amd.gen.generate import generate
        generate(build.GEN)
    body = kernels(compiled(source, tmp_path), f"comb_{planes}_strassen_{dtype}").popitem()[1]
    loads = re.findall(r"@llvm\.amdgcn\.raw\.ptr\.buffer\.load\.\w+\(.*, i32 (\d+)\)", body)
    assert len(loads) == 7 and set(loads) == policies, loads
