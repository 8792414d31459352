"""The launches of bf16 passes that cut some chains in two, as the C library issues them (CPU: a child process in
which the runtime's launch functions are stand-ins that record and, when told, refuse)."""
import os
import shutil
import subprocess
import sys

import pytest

import paper_2307_14995_amd as ltn

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2307_14995_amd", "libltn_attn.so")

STAND_INS = r"""
extern "C" {
struct Dim3 { unsigned x, y, z; };
static Dim3 grid_, block_;
static unsigned long shared_;
static void* stream_;
static int error_;
int launches, refuse_from = 1 << 30;           // launches asked for; the first that is refused
unsigned grids[16];
int __hipPushCallConfiguration(Dim3 g, Dim3 b, unsigned long s, void* st) { grid_ = g; block_ = b; shared_ = s; stream_ = st; return 0; }
int __hipPopCallConfiguration(Dim3* g, Dim3* b, unsigned long* s, void** st) { *g = grid_; *b = block_; *s = shared_; *st = stream_; return 0; }
int hipLaunchKernel(const void*, Dim3 g, Dim3, void**, unsigned long, void*) {
    if (launches < 16) grids[launches] = g.x;
    if (launches++ >= refuse_from) return error_ = 719;
    return 0;
}
int hipGetLastError() { const int e = error_; error_ = 0; return e; }
}
"""

CHILD = r"""
import ctypes, sys
rt = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)          # before the library, so that it binds to these
lib = ctypes.CDLL(sys.argv[2])
vp, ci, cl = ctypes.c_void_p, ctypes.c_int, ctypes.c_longlong
lib.ltn_attn_bwd.argtypes = [vp] * 8 + [ci, ci, cl, ci, ci, ci, vp, ctypes.c_size_t, vp]
launches, refuse = ctypes.c_int.in_dll(rt, "launches"), ctypes.c_int.in_dll(rt, "refuse_from")
P = 1 << 44                                                # fake addresses: nothing runs
def bwd(refuse_from):
    launches.value, refuse.value = 0, refuse_from
    rc = lib.ltn_attn_bwd(*(P + (i << 32) for i in range(8)), 8, 12, 1999, 96, 0, 1, None, 0, None)
    return rc, launches.value
print(bwd(1 << 30), bwd(0), bwd(1), list((ctypes.c_uint * 16).in_dll(rt, "grids"))[:2])
"""


def test_the_pass_is_not_launched_when_the_flags_are_not_cleared(tmp_path):
    cxx = shutil.which(os.environ.get("CXX", "g++"))
    if not cxx:
        pytest.skip("no host compiler")
    ltn.load_library()                                     # (built, if it was not)
    src, rt = tmp_path / "stand_ins.cpp", str(tmp_path / "stand_ins.so")
    src.write_text(STAND_INS)
    subprocess.run([cxx, "-O1", "-fPIC", "-shared", str(src), "-o", rt], check=True)
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1", ROCR_VISIBLE_DEVICES="-1")       # (nothing can reach a GPU)
    r = subprocess.run([sys.executable, "-c", CHILD, rt, LIB], env=env, capture_output=True, text=True, timeout=120)
    # 96 chains x 3 passes of 96 features: 32 chains more than a round of 256 workgroups, in two parts each.
    # Both launches; the clearing refused (nothing more is launched); the pass refused
    assert r.returncode == 0, r.stderr[-2000:]
    assert r.stdout.split("\n")[0] == "(0, 2) (6, 1) (6, 2) [1, 320]"
