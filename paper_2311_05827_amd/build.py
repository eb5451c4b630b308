"""Build libaccept.so (HIP kernels + C ABI) for gfx950, in-tree, with hipcc.

Usage: ``python -m paper_2311_05827_amd.build`` or ``build()`` from Python.  The library
lands next to this file; it is git-ignored but travels with the working tree.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB_PATH = os.path.join(HERE, "libaccept.so")
NATIVE_PATH = os.path.join(HERE, "_native.so")  # csrc/native.cpp: the Python binding's calls
SOURCES = ["api.hip", "uniform.hip", "uniform_chip_f32.hip", "uniform_chip_bf16.hip", "mbq.hip"]

HIPCC_FLAGS = [
    "-O3",
    "--offload-arch=gfx950",
    "-std=c++17",
    "-fPIC",
    "-ffp-contract=off",           # the quantizer's multiply and add must stay two roundings
    "-fno-gpu-flush-denormals-to-zero",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # The encoder's work-queue atomic is issued by one lane and its answer is looked at an item
    # later; the atomic optimizer would rewrite it into a form that waits for the answer at once.
    "-mllvm", "-amdgpu-atomic-optimizer-strategy=None",
    # A kernel's first eight words of arguments are in registers when its wavefronts start, instead of a load from memory
    # away: 0.05 to 0.5 us a kernel (2000 x 512, channels-last, round trip 13.2 -> 12.7 us; held pass, 205 MB
    # 54.0 -> 53.5; 262144 values, scheme M 6.62 -> 6.54).  Sixteen words: the same.
    "-mllvm", "-amdgpu-kernarg-preload-count=8",
    "-Wall", "-Wno-unused-function", "-Wno-unknown-warning-option",
    "-I", os.path.join(ROOT, "include"),
    "-I", CSRC,
]


def hipcc_path():
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (looked at $HIPCC, /opt/rocm/bin/hipcc, PATH)")


def _compile(hipcc, src, obj):
    cmd = [hipcc] + HIPCC_FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    return src, r.returncode, (r.stdout + r.stderr), " ".join(cmd)


def torch_lib():
    import torch
    return os.path.join(os.path.dirname(torch.__file__), "lib")


def _run(cmd):
    try:
        r = subprocess.run(cmd, capture_output=True, text=True)
    except OSError as e:
        return "%s\n%s" % (" ".join(cmd), e)
    return "" if r.returncode == 0 else "%s\n%s" % (" ".join(cmd), r.stdout + r.stderr)


def _compile_native(obj):
    """The binding's host code, against the installed PyTorch's headers (no device code: plain g++).  Returns what failed."""
    import torch
    from torch.utils.cpp_extension import include_paths
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-Wall",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI)]
    for path in include_paths() + [sysconfig.get_paths()["include"]]:
        cmd += ["-isystem", path]
    return _run(cmd + ["-I", os.path.join(ROOT, "include"), "-c", os.path.join(CSRC, "native.cpp"), "-o", obj])


def build(verbose=True):
    """Compile every HIP source and link libaccept.so, then the binding's _native.so.  Always recompiles."""
    hipcc = hipcc_path()
    lib_path = LIB_PATH
    bdir = os.path.join(HERE, "_build")
    os.makedirs(bdir, exist_ok=True)
    objs = [os.path.join(bdir, s.replace(".hip", ".o")) for s in SOURCES]
    with ThreadPoolExecutor(max_workers=len(SOURCES) + 1) as ex:
        compiling_native = ex.submit(_compile_native, os.path.join(bdir, "native.o"))
        results = list(ex.map(lambda so: _compile(hipcc, so[0], so[1]), zip(SOURCES, objs)))
    for src, rc, out, cmd in results:
        noise = "packed-fp32-ops' is not a recognized feature"
        shown = "\n".join(l for l in out.splitlines() if noise not in l)
        if rc != 0:
            raise RuntimeError("hipcc failed on %s\n%s\n%s" % (src, cmd, out))
        if verbose and shown.strip():
            print(shown, file=sys.stderr)
    tmp = lib_path + ".tmp"
    link = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    r = subprocess.run(link, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed\n%s\n%s" % (" ".join(link), r.stdout + r.stderr))
    os.replace(tmp, lib_path)
    # The library serves every call without _native.so (the binding then goes through ctypes, in more host time), so
    # a machine without g++ or Python's headers still builds it.
    failed = compiling_native.result() or _run(
        ["g++", "-shared", "-o", NATIVE_PATH + ".tmp", os.path.join(bdir, "native.o"), "-L" + HERE, "-l:libaccept.so",
         "-L" + torch_lib(), "-ltorch_python", "-ltorch_cpu", "-lc10", "-Wl,-rpath,$ORIGIN"])
    if failed:
        if os.path.exists(NATIVE_PATH):
            os.remove(NATIVE_PATH)  # an older one would be loaded
        print("not built: %s\n%s" % (NATIVE_PATH, failed), file=sys.stderr)
    else:
        os.replace(NATIVE_PATH + ".tmp", NATIVE_PATH)
    if verbose:
        print("built", lib_path, "" if failed else "and " + NATIVE_PATH, file=sys.stderr)
    return lib_path


if __name__ == "__main__":
    build()
