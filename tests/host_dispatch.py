"""The host side of the library with launchers that record instead of launching: which kernels a call would run, with which
arguments, found out on the CPU.  Pointers are never followed, so any aligned address stands for a matrix."""
import ctypes
import glob
import os
import re
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_06057_amd", "csrc")
GEN = os.path.join(CSRC, "generated")
DTYPES = {"f32": 0, "bf16": 1, "f16": 2}

STUBS = """
#include "lcma_params.h"
#include <string>
static thread_local std::string g_log;
extern "C" void dispatch_clear() { g_log.clear(); }
extern "C" const char *dispatch_log() { return g_log.c_str(); }
static int note(const char *name, const std::string &args = "") { g_log += std::string(name) + args + "\\n"; return 0; }
static std::string num(const char *k, long long v) { return std::string(" ") + k + "=" + std::to_string(v); }
static thread_local long long g_panel, g_rows; // of the last launch: column panels in tiles; rows of a plane (0: no batch)
extern "C" long long dispatch_panel() { return g_panel; }
extern "C" long long dispatch_plane_rows() { return g_rows; }
static std::string args(const lcma::PlaneGemmParams *p) {
    g_panel = p->panel;
    g_rows = p->c_plane / p->ldc_b;
    return num("jobs", p->jobs) + num("units", p->units) + num("ny", p->ny) + num("tail", p->tail_b) + num("panel", p->panel) + num("dealt", p->interleave);
}
static std::string args(const lcma::FewRowsParams *p) {
    g_panel = p->panel;
    return num("tile", p->block_rows) + num("steps", p->steps) + num("slices", p->slices) + num("slice_steps", p->slice_steps) + num("deep", p->deep);
}
static std::string args(const lcma::CombHParams *p) { return num("lanes", 1 << p->lane_shift) + num("streamed", p->streamed); }
"""

_lib = None


def lib():
    """Compiles the stub library (once per process) and returns it."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(os.path.join(GEN, "registry.cc")):
        from paper_2605_06057_amd.gen.generate import generate
        generate(GEN)
    host = [os.path.join(CSRC, f) for f in ("api.cc", "scheme.cc", "model.cc", "unfused.cc", "fp8_api.cc", "plane_gemm.cc")] + [os.path.join(GEN, "registry.cc")]
    out = tempfile.mkdtemp(prefix="lcma_dispatch_")
    objs = []
    procs = []
    for src in host:
        objs.append(os.path.join(out, os.path.basename(src) + ".o"))
        procs.append(subprocess.Popen(["g++", "-std=c++17", "-O1", "-fPIC", "-I", CSRC, "-I", GEN, "-c", src, "-o", objs[-1]]))
    assert all(p.wait() == 0 for p in procs)
    names = sorted(set(re.findall(r"\bU (lcma_launch_\w+)", subprocess.run(["nm"] + objs, check=True, capture_output=True, text=True).stdout)))
    stub = os.path.join(out, "stubs.cc")
    with open(stub, "w") as f:
        f.write(STUBS)
        for n in names:
            kind = ("FewRowsParams" if "few_rows" in n else "PlaneGemmParams" if n.startswith(("lcma_launch_pg_", "lcma_launch_pp")) else
                    "CombHParams" if "_comb_h" in n else None)
            f.write(f'extern "C" int {n}(const lcma::{kind} *p) {{ return note("{n[12:]}", args(p)); }}\n' if kind else
                    f'extern "C" int {n}() {{ return note("{n[12:]}"); }}\n')
    so = os.path.join(out, "dispatch.so")
    # (the buffer in the device image, lcma_static.hip, and its like are not needed here)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-I", CSRC, stub] + objs + ["-Wl,-Bsymbolic", "-o", so])
    L = ctypes.CDLL(so)
    for p in glob.glob(os.path.join(out, "*")):
        os.unlink(p)
    os.rmdir(out)
    L.dispatch_log.restype = L.lcma_last_error.restype = ctypes.c_char_p
    L.lcma_split_group_scratch_bytes.restype = L.dispatch_panel.restype = L.dispatch_plane_rows.restype = ctypes.c_int64
    _lib = L
    return L


A, B, C, WORK = 1 << 40, 2 << 40, 3 << 40, 4 << 40   # "device" addresses


class Scheme:
    def __init__(self, name):
        self.handle = ctypes.c_void_p()
        assert lib().lcma_scheme_load(f"builtin:{name}".encode(), ctypes.byref(self.handle)) == 0


def call(fn, *args):
    """(status, [launches]) of a call; ints are passed as int64 except those given as ctypes values."""
    L = lib()
    L.dispatch_clear()
    conv = [ctypes.c_int64(a) if isinstance(a, int) else a.handle if isinstance(a, Scheme) else a for a in args]
    status = getattr(L, fn)(*conv)
    return status, L.dispatch_log().decode().split("\n")[:-1]


def gemm(M, N, K, dtype, scheme=None, nk=False, ld=0):
    """lcma_gemm or (nk) lcma_gemm_nt of dense matrices, or with `ld` unused columns behind every row."""
    return call("lcma_gemm_nt" if nk else "lcma_gemm", M, N, K, A, K + ld, B, (K if nk else N) + ld, C, N + ld, ctypes.c_int(DTYPES[dtype]),
                Scheme(scheme) if scheme else ctypes.c_void_p(None), ctypes.c_void_p(None))


def gemm_prepared(M, N, K, dtype, scheme):
    return call("lcma_gemm_prepared", M, N, K, A, K, B, C, N, ctypes.c_int(DTYPES[dtype]), Scheme(scheme), ctypes.c_void_p(None))


def gemm_nt_ws(M, N, K, dtype, workspace_bytes, lda=None):
    return call("lcma_gemm_nt_ws", M, N, K, A, lda or K, B, K, C, N, ctypes.c_int(DTYPES[dtype]), WORK if workspace_bytes else 0, workspace_bytes,
                ctypes.c_void_p(None))
