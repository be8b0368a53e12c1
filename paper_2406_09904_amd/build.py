"""Builds libqqq.so (hand-written gfx950 kernels + the C ABI) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libqqq.so")
SOURCES = ["qqq_api.hip", "qqq_pack.hip", "qqq_quant_act.hip", "qqq_gemm_skinny.hip",
           "qqq_gemm_prefill_dma.hip", "qqq_gemm_prefill_ring.hip", "qqq_group_bias.hip", "qqq_quant_weight.hip", "qqq_probes.hip", "qqq_calib.hip",
           "qqq_hessian.hip", "qqq_compensate.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.sep not in c or os.path.exists(c)):
            return c
    raise RuntimeError("hipcc not found")


def call_path() -> str:
    """The linear calls' native marshalling (a Python extension), by the interpreter and the torch that it is built against: another's is never loaded."""
    import sysconfig

    import torch
    return os.path.join(HERE, "_qqq_call.torch-%s.%s.so" % (torch.__version__, sysconfig.get_config_var("SOABI")))


def build_call() -> str:
    """Compiles the Python extension against this interpreter and torch; returns its path."""
    import sysconfig

    import torch
    target = call_path()
    base = os.path.join(os.path.dirname(torch.__file__))
    inc = os.path.join(base, "include")
    tmp = target + ".tmp.%d" % os.getpid()
    # NDEBUG: pybind11 keeps a thread-local counter without it.  A library with a thread-local variable of its own that nothing reads makes every other
    # library's (torch's, HIP's) slower from its loading on, glibc looking through all of them at each access: two ctypes calls 14.5 -> 16.8 us.
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-DNDEBUG", "-I", sysconfig.get_paths()["include"], "-isystem", inc,
           "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"),
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), os.path.join(CSRC, "qqq_torch_call.cpp"), "-o", tmp,
           "-L", os.path.join(base, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed for qqq_torch_call.cpp:\n" + r.stdout + r.stderr)
    os.replace(tmp, target)
    return target


def build(verbose: bool = False, extra_flags=(), out_dir: str = None) -> str:
    """Compile every HIP source for gfx950 and link the shared library; returns its path.
    out_dir: build somewhere else (objects and library), e.g. a host-sanitizer build for the tests."""
    objdir = os.path.join(out_dir or HERE, "_build")
    lib_path = os.path.join(out_dir, "libqqq.so") if out_dir else LIB
    os.makedirs(objdir, exist_ok=True)
    cc = hipcc()

    def one(src):
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        cmd = [cc, *FLAGS, *extra_flags, "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        out = "\n".join(l for l in (r.stdout + r.stderr).splitlines()
                        if "packed-fp32-ops" not in l)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed for %s:\n%s" % (src, out))
        if verbose and out.strip():
            print(out, file=sys.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES) + 1)) as ex:
        call = ex.submit(build_call) if out_dir is None else None
        objs = list(ex.map(one, SOURCES))
        if call is not None:
            call.result()
    tmp = lib_path + ".tmp.%d" % os.getpid()
    r = subprocess.run([cc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout + r.stderr)
    os.replace(tmp, lib_path)
    return lib_path


if __name__ == "__main__":
    print(build(verbose=True))
