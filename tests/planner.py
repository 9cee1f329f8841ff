"""What the planner takes for a contraction, from csrc/plan.cpp compiled for the host
(tests/host_replay/dispatch.cpp)."""
import os
import shutil
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2007_08056_amd", "csrc")
ROCM_INCLUDE = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")
TUNING = ("SYMT_FUSED_V", "SYMT_GEMM_TILE", "SYMT_GEMM_SK", "SYMT_BF16_IL", "SYMT_BF16_FA")
F64, F32, C128, C64 = 0, 1, 2, 3
COMPUTE = {"f64": 0, "f32": 1, "bf16x3": 2}
STEPS = 0x100
_EXE = {}


def _exe():
    if "path" not in _EXE:
        gxx = shutil.which(os.environ.get("CXX", "g++"))
        if gxx is None or not os.path.isdir(ROCM_INCLUDE):
            pytest.skip("needs g++ and the ROCm headers")
        _EXE["dir"] = tempfile.TemporaryDirectory()
        path = os.path.join(_EXE["dir"].name, "dispatch")
        r = subprocess.run([gxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", ROCM_INCLUDE,
                            "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                            os.path.join(ROOT, "tests", "host_replay", "dispatch.cpp"), os.path.join(CSRC, "plan.cpp"),
                            "-o", path], capture_output=True, text=True, timeout=600)
        assert r.returncode == 0, r.stdout + r.stderr
        _EXE["path"] = path
    return _EXE["path"]


def line(sub, orders, su, du, sv, dv, dtype, compute, w=None, cu=0, cv=0, hu=None, hv=None, steps=False):
    """One contraction of operands in `dtype` (and w in `w`, by default the same; -1: none)."""
    fmt = lambda xs: ",".join(map(str, xs)) if xs else "-"
    return " ".join(map(str, (sub, fmt(orders), su, cu, fmt(du), fmt(hu), sv, cv, fmt(dv), fmt(hv), dtype, dtype,
                              dtype if w is None else w, COMPUTE[compute] | (STEPS if steps else 0))))


def plans(lines, **tuning):
    """The planner's choices (a dict of ints, or {"error": code}) for `lines`, under tuning variables."""
    env = {k: v for k, v in os.environ.items() if k not in TUNING}
    r = subprocess.run([_exe()], input="\n".join(lines) + "\n", capture_output=True, text=True, timeout=300,
                       env=dict(env, **tuning))
    assert r.returncode == 0, r.stderr
    return [{k: int(v) for k, v in (kv.split("=") for kv in ln.split())} for ln in r.stdout.splitlines()]
