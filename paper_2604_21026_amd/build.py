"""Build libnvq.so (gfx950 only) in-tree with hipcc, and _calls.so, the binding of the calls that
count in latency, with the host compiler against torch's headers.

    python -m paper_2604_21026_amd.build [--force]

Objects go to paper_2604_21026_amd/_build/ (git-ignored); the shared library
lands next to this file so that it travels with the source tree.
"""
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libnvq.so")
CALLS = os.path.join(HERE, "_calls.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ROCM = os.path.dirname(os.path.dirname(HIPCC)) or "/opt/rocm"
CXX = os.environ.get("CXX", "g++")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
    "-ffp-contract=off",
    # packed-fp32 instructions are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
]
# MFMA results go to ordinary vector registers (no accumulator-register copies), except in the
# prefill GEMM, whose accumulators alone fill the 256 ordinary registers of a wave
VGPR_FORM = ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]
NO_VGPR_FORM = {"gemm_w4a16.hip"}


def sources():
    return sorted(f for f in os.listdir(CSRC) if f.endswith(".hip"))


def _newest_header():
    hs = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".h")]
    hs.append(os.path.join(ROOT, "include", "nvq.h"))
    return max(os.path.getmtime(h) for h in hs)


def _compile(src, force, extra):
    obj = os.path.join(OBJ, src[:-4] + ".o")
    spath = os.path.join(CSRC, src)
    if (not force and os.path.exists(obj)
            and os.path.getmtime(obj) >= max(os.path.getmtime(spath), _newest_header())):
        return obj
    form = [] if src in NO_VGPR_FORM else VGPR_FORM
    subprocess.run([HIPCC] + FLAGS + form + list(extra) + ["-c", spath, "-o", obj], check=True)
    return obj


def _build_calls(force):
    src = os.path.join(CSRC, "binding.cpp")
    import torch
    # what the file was built for, besides the sources
    made_for, stamp = "torch %s python %s\n" % (torch.__version__, sys.version), os.path.join(OBJ, "calls.stamp")
    if (not force and os.path.exists(CALLS) and os.path.exists(stamp) and open(stamp).read() == made_for
            and os.path.getmtime(CALLS) >= max(os.path.getmtime(src), _newest_header())):
        return
    from torch.utils import cpp_extension
    inc = cpp_extension.include_paths() + [sysconfig.get_paths()["include"], os.path.join(ROCM, "include")]
    abi = int(torch._C._GLIBCXX_USE_CXX11_ABI)
    subprocess.run([CXX, "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM",
                    "-D_GLIBCXX_USE_CXX11_ABI=%d" % abi, '-DNVQ_TORCH_VERSION="%s"' % torch.__version__,
                    "-I" + os.path.join(ROOT, "include")]
                   + [a for i in inc for a in ("-isystem", i)] + [src, "-o", CALLS]
                   + ["-L" + d for d in cpp_extension.library_paths()]
                   + ["-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"], check=True)
    with open(stamp, "w") as f:
        f.write(made_for)


def build(force: bool = False, extra=()) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as ex:
        calls = ex.submit(_build_calls, force)
        objs = list(ex.map(lambda s: _compile(s, force, extra), sources()))
        subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs,
                       check=True)
        calls.result()  # (last: the library works without it)
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv))
