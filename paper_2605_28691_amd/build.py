"""Compiles the sources under csrc/ in-tree: libskiparse.so, the attention library, and libskiparse_probe.so, the measurement
micro-kernels the benchmark times (HIP, gfx950 only), and the module _marshal, the binding's native calls (host C++)."""
from __future__ import annotations

import glob
import importlib
import os
import subprocess
import sysconfig
import warnings

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libskiparse.so")
SOURCES = ["api.hip", "permute.hip", "attn_fwd.hip", "attn_bwd.hip", "attn_bwd_chain.hip", "quant_fp8.hip", "attn_fwd_fp8.hip"]
MARSHAL = os.path.join(HERE, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))  # found by the Python that it is built for
PROBE_LIB = os.path.join(HERE, "libskiparse_probe.so")
PROBE_SOURCES = ["mfma_probe.hip"]
FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-shared",
    # packed-fp32 instructions are kept out of the generated code on purpose
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def build(verbose: bool = False, save_temps: bool = False) -> str:
    """Builds everything; returns the path of the attention library."""
    _build_one(PROBE_LIB, PROBE_SOURCES, verbose, False)
    for old in glob.glob(os.path.join(HERE, "_marshal*.so")):  # never an old module beside a new library
        os.remove(old)
    _build_one(LIB, SOURCES, verbose, save_temps)
    try:
        _build_marshal(verbose)
    except (OSError, RuntimeError) as e:  # no host compiler, or no headers of this Python or torch
        warnings.warn(f"the native module of the binding was not built, calls go through ctypes: {e}")
    importlib.invalidate_caches()
    return LIB


def _build_marshal(verbose: bool) -> str:
    """The CPython module, compiled against torch's headers."""
    import torch

    from . import _torch_build

    root = os.path.dirname(torch.__file__)
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DBUILT_FOR="{_torch_build()}"',
           "-isystem", os.path.join(root, "include"), "-isystem", os.path.join(root, "include", "torch", "csrc", "api", "include"),
           "-isystem", sysconfig.get_paths()["include"],
           os.path.join(CSRC, "marshal.cpp"), "-o", MARSHAL + ".tmp",
           "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    _run(cmd, verbose)
    os.replace(MARSHAL + ".tmp", MARSHAL)
    return MARSHAL


def _build_one(lib: str, sources, verbose: bool, save_temps: bool) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc] + FLAGS + os.environ.get("SKIPARSE_EXTRA_FLAGS", "").split()
    if save_temps:
        tmp = os.path.join(HERE, "_build")
        os.makedirs(tmp, exist_ok=True)
        cmd += ["-save-temps=obj"]
        out = os.path.join(tmp, os.path.basename(lib))
    else:
        out = lib + ".tmp"
    cmd += ["-o", out] + [os.path.join(CSRC, s) for s in sources]
    _run(cmd, verbose)
    os.replace(out, lib)
    return lib


def _run(cmd, verbose: bool) -> None:
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass does not know the packed-fp32 target feature and says so; that is harmless
    log = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(os.path.basename(cmd[0]) + " failed:\n" + log)
    if verbose and log.strip():
        print(log)


if __name__ == "__main__":
    print(build(verbose=True, save_temps=bool(os.environ.get("SAVE_TEMPS"))))
