"""Which LM-head kernel and row shape the library takes for a problem: the library's own rule
(csrc/route.h), compiled for the host."""
import ctypes
import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@functools.lru_cache(None)
def _lib():
    with tempfile.TemporaryDirectory() as tmp:
        so = os.path.join(tmp, "route.so")
        subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC",
                               "-I", os.path.join(ROOT, "paper_2608_12913_amd", "csrc"),
                               os.path.join(ROOT, "tests", "native", "route_capi.cpp"), "-o", so])
        return ctypes.CDLL(so)


def route(rows, vocab, dp, dq, dtype="bf16", theta=0.1):
    """("stream", rows per workgroup) or ("wide", row blocks per wave)."""
    r = _lib().dcd_test_route(rows, vocab, dp, dq, int(dtype == "bf16"), int(theta == 0.0))
    return ("stream", r) if r > 0 else ("wide", -r)


def route_of(case, theta=None):
    return route(case.R, case.V, case.dp, case.dq, case.dtype, case.theta if theta is None else theta)
