"""Build step: compile the gfx950 HIP sources into paper_2307_14995_amd/libltn_attn.so.

hipcc cross-compiles for gfx950 without a GPU.  The library is built in-tree so that
it travels with the source tree; it is never installed elsewhere.  Every source is
compiled to an object of its own (in parallel), then linked; the compiler's per-kernel
resource report is read back and the build fails if a kernel that relies on registers
staying put (see ``NO_SPILL``) was given scratch memory or spilled vector registers.
Beside it goes the binding's native marshalling, paper_2307_14995_amd/_ltn_torch.so (host
code against torch's headers; it calls the library through addresses it is handed).
"""
from __future__ import annotations

import glob
import hashlib
import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libltn_attn.so")
TORCH_SRC = os.path.join(CSRC, "ltn_torch.cpp")
TORCH_LIB = os.path.join(PKG, "_ltn_torch.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep the compiler from forming packed-fp32 VALU ops
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # a kernel's first scalar arguments (14 words) in registers at its start: decode of 256 chains of 128 x 128 5.17 -> 4.86 us a
    # call, gate of 65536 rows 8.90 -> 8.72, the passes' scans; up to 128 chains, which the host bounds, nothing.  (Structs,
    # the passes' arguments, are loaded as before.)
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wno-unused-command-line-argument",
    "-Rpass-analysis=kernel-resource-usage",
]

# Kernels whose inline-assembly loads land in registers asynchronously (issued blocks ahead,
# waited for with explicit vmcnt counts): a spill or a stack copy between issue and wait would
# read stale data without any diagnostic, so such a build is refused.
NO_SPILL = re.compile(r"pass_bf16_kernel|tiled_(fwd|bwd)_bf16_kernel")


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _headers():
    return glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(ROOT, "include", "*.h"))


# Host-side sanitizer build (a checker's build, never what the product loads): AddressSanitizer and
# UndefinedBehaviorSanitizer on the host code only -- argument validation, plan selection, launch
# wrappers -- with the device code compiled as usual.
SAN_OBJ = os.path.join(PKG, "_build_san")
SAN_LIB = os.path.join(SAN_OBJ, "libltn_attn_san.so")
SAN_FLAGS = ["-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
             "-Xarch_host", "-fno-omit-frame-pointer", "-Xarch_host", "-fno-sanitize-recover=undefined"]


def _obj_of(src: str, objdir=None) -> str:
    return os.path.join(objdir or OBJ, os.path.basename(src) + ".o")


def _stale(target: str, deps) -> bool:
    if not os.path.exists(target):
        return True
    t = os.path.getmtime(target)
    return any(os.path.getmtime(d) > t for d in deps)


def _flags_of(extra=()) -> str:
    return " ".join(HIPCC_FLAGS + list(extra))


def _obj_stale(src: str, objdir=None, extra=()) -> bool:
    """Older than its source or a header, or compiled with other flags."""
    obj = _obj_of(src, objdir)
    if _stale(obj, [src] + _headers()) or not os.path.exists(obj + ".flags"):
        return True
    with open(obj + ".flags") as f:
        return f.read() != _flags_of(extra)


def marshalling_id() -> str:
    """What the native marshalling is built against: torch, the interpreter and the library's header."""
    import torch
    with open(os.path.join(ROOT, "include", "ltn_attn.h"), "rb") as f:
        header = hashlib.sha256(f.read()).hexdigest()[:16]
    return f"torch {torch.__version__} python {sys.version_info[0]}.{sys.version_info[1]} header {header}"


def marshalling_is_stale() -> bool:
    if _stale(TORCH_LIB, [TORCH_SRC] + _headers()):
        return True
    with open(TORCH_LIB, "rb") as f:
        return marshalling_id().encode() not in f.read()


def is_stale() -> bool:
    return _stale(LIB, sources() + _headers()) or any(_obj_stale(s) for s in sources()) or marshalling_is_stale()


def check_resource_report(report: str) -> None:
    """Raise if a NO_SPILL kernel of this compiler report uses scratch or spilled VGPRs."""
    bad = []
    name = None
    for line in report.splitlines():
        m = re.search(r"remark: Function Name: (\S+)", line)
        if m:
            name = m.group(1)
            continue
        m = re.search(r"remark:\s+(ScratchSize \[bytes/lane\]|VGPRs Spill): (\d+)", line)
        if m and name and NO_SPILL.search(name) and int(m.group(2)) != 0:
            bad.append(f"{name}: {m.group(1)} = {m.group(2)}")
    if bad:
        raise RuntimeError("kernels with register-resident asynchronous loads must not spill:\n  " + "\n  ".join(bad))


def _compile(src: str, hipcc: str, verbose: bool, objdir=None, extra=()) -> str:
    obj = _obj_of(src, objdir)
    if os.path.exists(obj + ".flags"):                 # (a compilation that fails leaves no record for the old object)
        os.remove(obj + ".flags")
    cmd = [hipcc] + HIPCC_FLAGS + list(extra) + ["-I", os.path.join(ROOT, "include"), "-c", src, "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n" + res.stdout + res.stderr)
    check_resource_report(res.stderr)
    with open(obj + ".flags", "w") as f:
        f.write(_flags_of(extra))
    with open(obj + ".resources.txt", "w") as f:       # kept beside the object for inspection
        f.write("\n".join(l for l in res.stderr.splitlines() if "remark:" in l and "Function Name" in l or
                          re.search(r"remark:\s+(VGPRs|AGPRs|ScratchSize|Occupancy|VGPRs Spill|SGPRs Spill|LDS Size)", l)))
    return obj


def build_marshalling(verbose: bool = False) -> str:
    """Compile the binding's native marshalling against the installed torch.  It takes its place in one
    step: a process that starts meanwhile finds the old file, the new one or none, never half of one."""
    import sysconfig

    import torch
    root = os.path.dirname(torch.__file__)
    include, lib = os.path.join(root, "include"), os.path.join(root, "lib")
    tmp = f"{TORCH_LIB}.{os.getpid()}.tmp"
    cmd = [os.environ.get("CXX", "g++"), f'-DLTN_BUILT_FOR="{marshalling_id()}"', "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-isystem", include,
           "-isystem", os.path.join(include, "torch", "csrc", "api", "include"), "-isystem", "/opt/rocm/include",
           "-isystem", sysconfig.get_paths()["include"], TORCH_SRC, "-o", tmp, "-L", lib, "-ltorch_python",
           "-ltorch_cpu", "-lc10", "-lc10_hip"]
    if verbose:
        print(" ".join(cmd), flush=True)
    try:
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError(f"{cmd[0]} failed on {TORCH_SRC}:\n" + res.stdout + res.stderr)
        os.replace(tmp, TORCH_LIB)
    finally:
        if os.path.exists(tmp):
            os.remove(tmp)
    return TORCH_LIB


def build_library(force: bool = True, verbose: bool = False, marshalling: bool = True) -> str:
    """Compile every HIP source for gfx950 (all of them when `force`, otherwise only those
    older than a source or header or compiled with other flags), link the shared library, and build the marshalling beside it
    (a failure there is raised once the library is complete)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ, exist_ok=True)
    srcs = sources()
    todo = [s for s in srcs if force or _obj_stale(s)]
    jobs = int(os.environ.get("MAX_JOBS", "8") or 8)
    with ThreadPoolExecutor(max_workers=max(1, min(jobs, 16))) as pool:
        beside = pool.submit(build_marshalling, verbose) if marshalling and (force or marshalling_is_stale()) else None
        list(pool.map(lambda s: _compile(s, hipcc, verbose), todo))
    objs = [_obj_of(s) for s in srcs]
    if todo or _stale(LIB, objs):
        cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", LIB]
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError("link failed:\n" + res.stdout + res.stderr)
    if beside:
        beside.result()
    return LIB


def sanitizer_runtime() -> str:
    """Path of the shared AddressSanitizer runtime of the compiler that hipcc drives."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    res = subprocess.run([hipcc, "-print-file-name=libclang_rt.asan-x86_64.so"], capture_output=True, text=True)
    path = res.stdout.strip()
    if not os.path.isabs(path):
        cands = glob.glob("/opt/rocm/lib/llvm/lib/clang/*/lib/linux/libclang_rt.asan-x86_64.so")
        path = cands[0] if cands else ""
    return path


def build_sanitized(verbose: bool = False) -> str:
    """The same sources with ASan + UBSan on the host code, linked against the shared sanitizer
    runtime, into _build_san/ (only what is stale is recompiled)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(SAN_OBJ, exist_ok=True)
    srcs = sources()
    todo = [s for s in srcs if _obj_stale(s, SAN_OBJ, SAN_FLAGS)]
    jobs = int(os.environ.get("MAX_JOBS", "8") or 8)
    with ThreadPoolExecutor(max_workers=max(1, min(jobs, 16))) as pool:
        list(pool.map(lambda s: _compile(s, hipcc, verbose, SAN_OBJ, SAN_FLAGS), todo))
    objs = [_obj_of(s, SAN_OBJ) for s in srcs]
    if todo or _stale(SAN_LIB, objs):
        cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-fsanitize=address", "-fsanitize=undefined",
               "-shared-libsan"] + objs + ["-o", SAN_LIB]
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError("sanitizer link failed:\n" + res.stdout + res.stderr)
    return SAN_LIB


if __name__ == "__main__":
    print(build_library(force="--stale-only" not in sys.argv, verbose=True))
