"""Compile the HIP sources under csrc/ into libla.so (gfx950 only) and the native part of the Python
binding into _marshal.so, in-tree."""
import glob
import os
import subprocess
import sys
import sysconfig
import warnings

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libla.so")
MARSHAL = os.path.join(HERE, "_marshal.so")

CXX = "g++"
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    "-fvisibility=hidden",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build_library(verbose=False, extra_flags=(), out=LIB):
    """Always recompiles; returns the path of the shared library."""
    cmd = [HIPCC] + FLAGS + list(extra_flags) + ["-I", INCLUDE, "-I", CSRC] + sources() + ["-o", out]
    if verbose:
        print(" ".join(cmd))
    subprocess.run(cmd, check=True)
    return out


def build_marshal(verbose=False, out=MARSHAL):
    """The argument marshalling of binding.py (host code, against torch's headers).  binding.py works without
    it: where it cannot be built, a warning says why, None is returned and no older file stays."""
    if os.path.exists(out):
        os.remove(out)
    try:
        return _compile_marshal(verbose, out)
    except (ImportError, OSError, subprocess.CalledProcessError) as e:
        warnings.warn("%s is not built, calls take a few microseconds longer: %s" % (out, e), RuntimeWarning,
                      stacklevel=2)


def _compile_marshal(verbose, out):
    import torch
    from torch.utils.cpp_extension import include_paths, library_paths
    cmd = [CXX, "-O2", "-std=c++17", "-shared", "-fPIC", "-fvisibility=hidden",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
           '-DLA_BUILT_FOR="torch %s, Python %d.%d"' % (torch.__version__, *sys.version_info[:2]), "-I", INCLUDE]
    cmd += ["-isystem%s" % p for p in include_paths() + [os.path.join(ROCM, "include"), sysconfig.get_paths()["include"]]]
    cmd += [os.path.join(CSRC, "la_bind.cpp")]
    cmd += ["-L%s" % p for p in library_paths()] + ["-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10", "-o", out]
    if verbose:
        print(" ".join(cmd))
    subprocess.run(cmd, check=True)
    return out


if __name__ == "__main__":
    print(build_library(verbose=True))
    print(build_marshal(verbose=True))
