"""Build libtbn.so (HIP for gfx950) and the Python binding in-tree with hipcc.

Every .hip/.cpp file under csrc/ is compiled to an object in _build/ (in parallel) and
linked into paper_1701_00485_amd/libtbn.so.  Packed-FP32 instruction selection is
disabled for all device code.  native/tbn_torch.cpp (host code against torch's headers)
becomes paper_1701_00485_amd/_tbn_torch.so, which finds libtbn.so beside it.
"""
from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libtbn.so")
BINDING = os.path.join(PKG, "_tbn_torch.so")
ARCH = os.environ.get("TBN_OFFLOAD_ARCH", "gfx950")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
COMMON = ["-O3", "-fPIC", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
          "-Wall", "-Wno-unused-function"]
DEVICE = ["-x", "hip", "--offload-arch=" + ARCH,
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".hip", ".cpp")))


def _compile(src):
    obj = os.path.join(BUILD, os.path.basename(src) + ".o")
    cmd = [HIPCC] + COMMON + DEVICE + ["-c", src, "-o", obj]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines()
                    if "packed-fp32-ops" not in l and "is not a recognized feature" not in l)
    if r.returncode != 0:
        raise RuntimeError("compile failed: %s\n%s" % (" ".join(cmd), out))
    return obj, out


def _compile_binding():
    import torch
    from torch.utils import cpp_extension

    src = os.path.join(PKG, "native", "tbn_torch.cpp")
    obj = os.path.join(BUILD, "tbn_torch.cpp.o")
    includes = [os.path.join(ROOT, "include"), sysconfig.get_paths()["include"]] + cpp_extension.include_paths()
    includes.append(os.path.join(os.path.dirname(os.path.dirname(HIPCC)), "include"))
    cmd = [HIPCC, "-x", "c++", "-O2", "-fPIC", "-std=c++17", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           '-DTBN_TORCH_VERSION="%s"' % torch.__version__]
    for i in includes:
        cmd += ["-isystem" if "torch" in i else "-I", i]
    r = subprocess.run(cmd + ["-c", src, "-o", obj], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("compile failed: %s\n%s" % (" ".join(cmd), r.stdout))
    return obj, r.stdout


def _link_binding(obj):
    from torch.utils import cpp_extension

    tmp = BINDING + ".tmp%d" % os.getpid()
    cmd = [HIPCC, "-shared", "-fPIC", "-o", tmp, obj, LIB, "-Wl,-rpath,$ORIGIN"]
    cmd += ["-L" + p for p in cpp_extension.library_paths()]
    subprocess.check_call(cmd + ["-lc10", "-ltorch_cpu", "-ltorch_python", "-lc10_hip"])
    os.replace(tmp, BINDING)


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    srcs = sources()
    with concurrent.futures.ThreadPoolExecutor(max_workers=8) as ex:
        binding = ex.submit(_compile_binding)
        results = list(ex.map(_compile, srcs))
        binding_obj = binding.result()[0]
    if verbose:
        for _, out in results:
            if out.strip():
                print(out)
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=" + ARCH, "-Wl,-soname,libtbn.so", "-o", tmp]
    subprocess.check_call(cmd + [o for o, _ in results])
    os.replace(tmp, LIB)
    _link_binding(binding_obj)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
