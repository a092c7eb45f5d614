"""Where the tile of C takes the place of the stages in LDS, its writes and reads lie outside the promise that the loop over K makes to the
compiler, namely that nothing else reaches the stages (restrict); under it the compiler may move them in front of the last reads
of a stage.  From the alias scopes of the compiler's own output."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2605_06057_amd import build


def compiled(source, tmp_path):
    """LLVM IR of the device code of a source."""
    out = str(tmp_path / "out.ll")
    subprocess.run([build.HIPCC] + build.COMMON + build.DEVICE_FLAGS + ["--cuda-device-only", "-S", "-emit-llvm", source, "-o", out], check=True, capture_output=True)
    return open(out).read()


def kernels(text, name):
    """{name: IR} of the kernels that match `name`."""
    return {m.group(1): m.group(0) for m in re.finditer(rf"^define [^\n]*@lcma_k_({name})\(.*?^}}", text, re.M | re.S)}


@pytest.mark.skipif(not (os.path.exists(build.HIPCC) or shutil.which(build.HIPCC)), reason="needs hipcc")
def test_partial_tiles_of_the_few_rows_kernels(tmp_path):
    text = compiled(os.path.join(build.CSRC, "lcma_few_rows.hip"), tmp_path)
    found = kernels(text, r"few_rows_b?f16_\w+")
    assert sorted(found) == sorted(f"few_rows_{t}_{n}" for t in ("bf16", "f16") for n in ("16", "16_deep", "32", "64"))
    for name, body in found.items():
        sums = re.findall(r"^.*(?:store float .*|load <4 x float>, )ptr addrspace\(3\).*$", body, re.M)
        assert sum("store" in line for line in sums) >= 4 and any("load" in line for line in sums), name
        assert "!noalias" in body, f"{name}: the loop has lost its promise"
        assert not [line for line in sums if "!noalias" in line or "!alias.scope" in line], name
    # A CU holds several work-groups of the smaller tiles: with 128 KB each 1 x 14336 x 1024 took 12.2 us, 7.6 with 32
    lds = {m.group(1): int(m.group(2)) for m in re.finditer(r"_few_rows_(b?f16_\w+?)E4smem = .*?\[(\d+) x i8\]", text)}
    for t in ("bf16", "f16"):
        assert lds[f"{t}_16"] <= 32768 and lds[f"{t}_32"] <= 65536 and lds[f"{t}_16_deep"] <= 131072, lds


def test_no_function_reaches_the_stages_by_both_ways():
    """A function that is handed the stages as restrict pointers gets no pointer to all of LDS besides: the 256 x 128 ping-pong kernel, which has both,
    makes no such promise (its compiled form carried no alias scopes before, so this is held in the source)."""
    import glob
    lists = [re.sub(r"\s+", " ", m.group(1)) for path in glob.glob(os.path.join(build.CSRC, "*.hpp")) for m in re.finditer(r"LCMA_DEV void \w+\(([^;{}]*?__restrict__[^;{}]*?)\) \{", open(path).read())]
    assert len(lists) >= 3
    for parameters in lists:
        assert not re.search(r"LCMA_LDS char \*(?!__restrict__)", parameters), parameters
