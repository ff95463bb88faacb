"""Build ``libzpp.so`` (the HIP kernels and the C ABI) for gfx950 and the
binding's ``_marshal.so`` in-tree.

    python -m paper_2407_01614_amd.build          # both, and libzpp_ceiling.so
"""
import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libzpp.so")
# the plain HBM streams that bench.py times beside the kernels (not the path)
CEILING_LIB = os.path.join(PKG, "libzpp_ceiling.so")
CEILING_SOURCES = ["ceiling.hip"]
# the Python binding's tensor marshalling (host code)
MARSHAL_LIB = os.path.join(PKG, "_marshal.so")
MARSHAL_SOURCE = "marshal.cpp"

SOURCES = ["zpp_api.hip", "adam.hip", "refresh.hip", "quant.hip", "gather.hip", "fused.hip",
           "qgz.hip", "receive_adam.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-shared",
    "-fvisibility=hidden",
    "-Wall",
    "-Werror",
    # IEEE fp32 division and square root, denormals kept: the quantization
    # codes and scales must be the correctly rounded binary32 results.
    "-fhip-fp32-correctly-rounded-divide-sqrt",
    "-fno-gpu-flush-denormals-to-zero",
    "-fno-fast-math",
    # no packed-fp32 VALU forms (v_pk_{add,mul,fma}_f32) in generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def hipcc():
    for cand in (os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc"), "hipcc"):
        if os.path.sep not in cand or os.path.exists(cand):
            return cand
    return "hipcc"


def build(out=LIB, defines=(), verbose=False, sources=SOURCES):
    """Compile the HIP sources of the path into one shared library; with the
    library itself, what its Python binding needs beside it (_marshal.so)."""
    tmp = out + ".tmp%d" % os.getpid()
    cmd = [hipcc(), *HIPCC_FLAGS, *["-D" + d for d in defines], "-I", INCLUDE, "-I", CSRC,
           *[os.path.join(CSRC, s) for s in sources], "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass does not know the packed-fp32 feature and says so; that
    # warning is expected, anything else is shown
    noise = "not a recognized feature for this target"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l and l.strip())
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + res.stderr)
    if err and verbose:
        print(err, file=sys.stderr)
    os.replace(tmp, out)
    if out == LIB:
        build_marshal(verbose=verbose)
    return out


def build_ceiling(verbose=False):
    """Compile the measurement streams into libzpp_ceiling.so."""
    return build(out=CEILING_LIB, verbose=verbose, sources=CEILING_SOURCES)


def build_marshal(verbose=False):
    """Compile the binding's tensor marshalling (host code against torch's
    headers) into _marshal.so."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    tmp = MARSHAL_LIB + ".tmp%d" % os.getpid()
    torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
           *[x for d in cpp_extension.include_paths() for x in ("-isystem", d)],
           "-isystem", sysconfig.get_paths()["include"],
           os.path.join(CSRC, MARSHAL_SOURCE), "-o", tmp,
           "-L" + torch_lib, "-ltorch_python", "-ltorch_cpu", "-lc10"]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("g++ failed:\n" + res.stderr)
    os.replace(tmp, MARSHAL_LIB)
    return MARSHAL_LIB


if __name__ == "__main__":
    print(build(verbose=True))
    print(build_ceiling(verbose=True))
