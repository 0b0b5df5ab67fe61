"""Builds libstc.so (HIP, gfx950 only) in-tree with hipcc."""
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

import torch

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG_DIR, "csrc")
LIB_PATH = os.path.join(PKG_DIR, "libstc.so")
BENCH_LIB_PATH = os.path.join(PKG_DIR, "libstc_bench.so")   # benchmark-only helpers (bench.py)
BINDING_PATH = os.path.join(PKG_DIR, "_binding.so")         # Python's way into libstc.so
BUILD_DIR = os.path.join(PKG_DIR, "_build")

SOURCES = ["stc_api.hip", "bounds.hip", "router.hip", "route_pack.hip", "flush.hip",
           "score.hip", "select.hip", "attention.hip", "step.hip"]

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC",
    # packed-FP32 VALU forms are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    # the first scalar arguments of a kernel (14 words at most) are in registers when it starts
    # instead of a load from memory away: 0.9 us per layer of a decode step of three launches
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
]
# matrix-core results are consumed by vector instructions right away, so keep them in
# ordinary vector registers (no copies out of the accumulation registers)
_VGPR_MFMA = ["-mllvm", "-amdgpu-mfma-vgpr-form"]
FILE_FLAGS = {"score.hip": _VGPR_MFMA, "attention.hip": _VGPR_MFMA, "step.hip": _VGPR_MFMA,
              "router.hip": _VGPR_MFMA}


def _hipcc():
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    return "hipcc"


def _binding_cmds(obj):
    """Compiling and linking csrc/binding.cpp: host code against the headers of the installed torch."""
    root, include = os.path.dirname(torch.__file__), sysconfig.get_path("include")
    compile_ = ["g++", "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden",
                "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
                "-I" + os.path.join(root, "include"),
                "-I" + os.path.join(root, "include", "torch", "csrc", "api", "include"),
                "-I" + include, "-c", os.path.join(CSRC, "binding.cpp"), "-o", obj]
    link = ["g++", "-shared", obj, "-o", BINDING_PATH, "-L" + os.path.join(root, "lib"),
            "-ltorch_python", "-ltorch_cpu", "-lc10", "-L" + PKG_DIR, "-lstc", "-Wl,-rpath,$ORIGIN"]
    return compile_, link


def _run(cmd):
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("command failed: %s\n%s" % (" ".join(cmd), r.stdout))
    return r.stdout


def build_library(verbose=False):
    """Compile every source, link libstc.so and Python's way into it; always recompiles."""
    os.makedirs(BUILD_DIR, exist_ok=True)
    hipcc = _hipcc()
    objs = [os.path.join(BUILD_DIR, s.replace(".hip", ".o")) for s in SOURCES]

    def one(pair):
        src, obj = pair
        out = _run([hipcc, *HIPCC_FLAGS, *FILE_FLAGS.get(src, []), "-c",
                    os.path.join(CSRC, src), "-o", obj])
        if verbose and out.strip():
            print(out)

    compile_binding, link_binding = _binding_cmds(os.path.join(BUILD_DIR, "binding.o"))
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        binding = ex.submit(_run, compile_binding)
        list(ex.map(one, zip(SOURCES, objs)))
        binding.result()
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB_PATH, *objs])
    _run([hipcc, *HIPCC_FLAGS, "-shared", "-o", BENCH_LIB_PATH,
          os.path.join(CSRC, "bench_stream.hip")])
    _run(link_binding)
    return LIB_PATH


if __name__ == "__main__":
    print(build_library(verbose="-v" in sys.argv))
