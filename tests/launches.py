"""Which kernels an entry point launches, found without a GPU: a process of its own makes the calls with launch_recorder.cpp in the
place of the HIP runtime's launch."""
import functools
import json
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
P = 1 << 20  # an aligned address that nothing reads

CHILD = """
import ctypes, json, sys
sys.path.insert(0, sys.argv[1])
recorder = ctypes.CDLL(sys.argv[2], mode=ctypes.RTLD_GLOBAL)  # before the library, which then finds its hipLaunchKernel here
recorder.recorded.restype = ctypes.c_char_p
from paper_2307_08691_amd import binding
out = []
for name, args in json.load(sys.stdin):
    status = getattr(binding, name + "_raw")(*args)
    lines = [l.split("|") for l in recorder.recorded().decode().splitlines()]
    out.append([status, [[k.split("fa::", 1)[1].rsplit("(", 1)[0], int(x), int(y), int(t)] for k, x, y, t in lines]])
json.dump(out, sys.stdout)
"""


@functools.lru_cache(None)
def recorder():
    so = os.path.join(tempfile.mkdtemp(prefix="fa_launches_"), "recorder.so")
    subprocess.run([os.environ.get("CXX", "g++"), "-O1", "-std=c++17", "-shared", "-fPIC", "-o", so,
                    os.path.join(HERE, "launch_recorder.cpp"), "-ldl"], check=True)
    return so


def launches(calls):
    """[(entry point, arguments of its _raw form)] -> per call the kernels in order: (name, workgroups x, workgroups y, threads)."""
    r = subprocess.run([sys.executable, "-c", CHILD, ROOT, recorder()], input=json.dumps(calls), capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    out = json.loads(r.stdout)
    assert all(status == 0 for status, _ in out), [s for s, _ in out]
    return [[tuple(k) for k in kernels] for _, kernels in out]


def varlen_cross_bwd(nseq, total_q, total_k, max_q, max_k, Hq, Hkv, d, causal=False, f16=False):
    return "fa_varlen_cross_bwd", [P] * 10 + [1 << 40, P, P, nseq, total_q, total_k, max_q, max_k, Hq, Hkv, d, 0.1, causal, 0, f16]


def cross_bwd(B, Hq, Hkv, Nq, Nk, d, causal=False, f16=False):
    return "fa_cross_bwd", [P] * 10 + [1 << 40, B, Hq, Hkv, Nq, Nk, d, 0.1, causal, 0, f16]


def mask_bwd(B, Hq, Hkv, Nq, Nk, d, causal=False, f16=False):
    return "fa_mask_bwd", [P] * 11 + [1 << 40, B, Hq, Hkv, Nq, Nk, d, 0.1, causal, 0, 0, (Nk + 7) // 8 * 8, 0, f16]


def dropout_bwd(B, Hq, Hkv, Nq, Nk, d, causal=False, f16=False):
    return "fa_dropout_bwd", [P] * 10 + [1 << 40, B, Hq, Hkv, Nq, Nk, d, 0.1, causal, 0.1, 7, 0, f16]


def varlen_bwd(nseq, total, longest, Hq, Hkv, d, workspace=1 << 40, causal=False):
    return "fa_varlen_bwd", [P] * 10 + [workspace, P, nseq, total, longest, Hq, Hkv, d, 0.1, causal, 0, False]
