"""Order of reads and loads at the start of the 256 x 256 ping-pong kernel (csrc/lcma_pingpong.hpp), from its assembly: every wave
reads half 0 of B before the first step, and the first load of that step goes to the same place in LDS, so a wait for the reads and a
barrier that ALL waves execute have to lie between (a race shows in no result that a test could rely on)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2605_06057_amd import build

SOURCE = """#include "lcma_pingpong.hpp"
#define KERNEL(NAME, ...) \\
    extern "C" __global__ __launch_bounds__(512, 2) void NAME(const lcma::PlaneGemmParams) { \\
        using G = lcma::PingPongGemm<__VA_ARGS__>; \\
        __shared__ __attribute__((aligned(16))) char smem[G::LDS_BYTES]; \\
        G::run((LCMA_LDS char *)smem); \\
    }
KERNEL(rows_bf16, lcma::BF16, lcma::BF16)
KERNEL(rows_f16_f32, lcma::F16, lcma::F32)
KERNEL(columns_bf16, lcma::BF16, lcma::BF16, true)
KERNEL(columns_f16, lcma::F16, lcma::F16, true)
KERNEL(fp8_bf16, lcma::FP8, lcma::BF16)
KERNEL(fp8_f16, lcma::FP8, lcma::F16)
"""


@pytest.mark.skipif(not (os.path.exists(build.HIPCC) or shutil.which(build.HIPCC)), reason="needs hipcc")
def test_first_reads_end_before_the_first_load_behind_them(tmp_path):
    src, out = tmp_path / "start.hip", tmp_path / "start.s"
    src.write_text(SOURCE)
    subprocess.run([build.HIPCC] + build.COMMON + build.DEVICE_FLAGS + ["--cuda-device-only", "-S", str(src), "-o", str(out)], check=True, capture_output=True)
    bodies = re.findall(r"^(\w+):\s+; @\1$(.*?)^\.Lfunc_end", out.read_text(), re.M | re.S)
    assert len(bodies) == 6
    for name, body in bodies:
        reads = waited = False
        for line in body.splitlines():
            op = line.split()
            if not op:
                continue
            if op[0].startswith("ds_read"):
                reads, waited = True, False
            elif not reads:
                continue
            elif op[0] == "s_waitcnt":
                waited |= "lgkmcnt(0)" in line
            elif op[0] == "s_barrier":
                assert waited, f"{name}: barrier in front of the end of the first reads"
                break
            # a branch or label: what follows is not executed by every wave
            assert not (op[0].startswith(("s_cbranch", "s_branch")) or op[0].startswith(".LBB") or "lds" in op[1:] and op[0].startswith("buffer_load")), \
                f"{name}: no barrier for all waves behind the first reads: {line.strip()}"
        else:
            pytest.fail(f"{name}: no barrier")
