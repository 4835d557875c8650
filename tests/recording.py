"""Runs the library's calls in a process of their own with the HIP runtime's host
calls replaced by tests/recording_runtime.cpp: nothing is launched, and what would
be is returned, as dicts of name, blocks, threads and status."""
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

CHILD = r"""
import ctypes as ct, json, sys
R = ct.CDLL(sys.argv[1], mode=ct.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
from paper_1908_06649_amd import tcu
L = tcu.lib()
for f, t in (("rec_name", ct.c_char_p), ("rec_blocks", ct.c_uint64), ("rec_threads", ct.c_uint32)):
    getattr(R, f).restype = t
P = [0x10000000000 + (i << 42) for i in range(8)]     # never dereferenced
out = []
for job in json.load(sys.stdin):
    for k, v in job.get("knobs", []):
        assert L.tcu_set_knob(k, v) == 0
    for part, n in job.get("arity", []):
        R.rec_arity(part.encode(), n)
    R.rec_reset(job.get("fail", -1))
    rc = getattr(L, job["fn"])(*[P[a["p"]] if isinstance(a, dict) else a for a in job["args"]])
    out.append({"rc": rc, "launches": [
        {"name": R.rec_name(i).decode(), "blocks": R.rec_blocks(i), "threads": R.rec_threads(i),
         "status": R.rec_status(i), "ints": [R.rec_int(i, a) for a in range(16)]}
        for i in range(R.rec_count())]})
    for k, v in job.get("knobs", []):
        assert L.tcu_set_knob(k, 0) == 0
print("RESULT" + json.dumps(out))
"""


def build(folder) -> str:
    so = os.path.join(str(folder), "recording_runtime.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    f"-I{ROCM}/include", "-o", so,
                    os.path.join(ROOT, "tests", "recording_runtime.cpp")], check=True)
    return so


def ptr(i: int) -> dict:
    """A device address, 16-byte aligned, far from the others."""
    return {"p": i}


def run(so: str, jobs) -> list:
    res = subprocess.run([sys.executable, "-c", CHILD, so, ROOT], input=json.dumps(jobs),
                         capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout + res.stderr
    return json.loads(res.stdout[res.stdout.index("RESULT") + 6:])


def product(M, K, N, dtype, *, lda=None, ldb=None, ldc=None, acc=False, knobs=(), **kw) -> dict:
    return dict(fn="tcu_gemm_rect_ex", knobs=list(knobs),
                args=[ptr(0), lda or K, ptr(1), ldb or N, ptr(2), ldc or N, M, K, N, int(acc), 16,
                      dtype, None], **kw)
