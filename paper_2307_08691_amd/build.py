"""Build the gfx950 attention library in-tree with hipcc, and the native marshalling of its binding with the C++ compiler.

    python -m paper_2307_08691_amd.build

produces paper_2307_08691_amd/libfa_gfx950.so from csrc/*.hip and paper_2307_08691_amd/_host.so from csrc/fa_host.cpp. hipcc
cross-compiles for gfx950 without a GPU.
"""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libfa_gfx950.so")
HOST_LIB = os.path.join(HERE, "_host.so")  # (a Python extension module)
SOURCES = ["fa_api.hip", "fa_fwd.hip", "fa_stream.hip", "fa_bwd.hip", "fa_joint64.hip", "fa_joint128.hip", "fa_shares64.hip", "fa_shares128.hip", "fa_short.hip", "fa_d256.hip", "fa_fp8.hip", "fa_decode.hip", "fa_probe.hip"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.sep not in c or os.path.exists(c)):
            return c
    raise RuntimeError("hipcc not found")


def _compile(source: str, obj: str) -> str:
    cmd = [hipcc(), *FLAGS, "-c", "-o", obj, os.path.join(CSRC, source)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass does not know the AMDGPU-only target feature and says so: harmless
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip())
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {source}:\n" + err)
    return err


def build_host() -> None:
    """Compile the extension module against the installed torch."""
    import sysconfig
    import torch
    from torch.utils import cpp_extension
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           *(f"-I{d}" for d in cpp_extension.include_paths() + [sysconfig.get_paths()["include"]]),
           "-o", HOST_LIB, os.path.join(CSRC, "fa_host.cpp"), f"-L{lib}", "-ltorch_python", "-ltorch_cpu", "-lc10"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("the C++ compiler failed on fa_host.cpp:\n" + r.stderr)


def build(verbose: bool = False) -> str:
    """Compile every HIP source (in parallel, one object each) and link the shared library.
    Always recompiles. The extension module is optional: without torch or a C++ compiler that takes it the library is built all
    the same, the reason is printed, and none is left from an earlier build (it would be older than the library)."""
    import concurrent.futures
    import tempfile
    with tempfile.TemporaryDirectory(prefix="fa_build_") as tmp:
        objs = [os.path.join(tmp, s.replace(".hip", ".o")) for s in SOURCES]
        if verbose:
            print(" ".join([hipcc(), *FLAGS, "-c"]), *SOURCES, flush=True)
        with concurrent.futures.ThreadPoolExecutor(len(SOURCES) + 1) as ex:
            host = ex.submit(build_host)
            for err in ex.map(_compile, SOURCES, objs):
                if verbose and err:
                    print(err, file=sys.stderr)
            try:
                host.result()
            except Exception as e:
                print(f"no {os.path.basename(HOST_LIB)}, the usual calls will be made in Python: {e}", file=sys.stderr)
                if os.path.exists(HOST_LIB):
                    os.remove(HOST_LIB)
        r = subprocess.run([hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs], capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("link failed:\n" + r.stderr)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
