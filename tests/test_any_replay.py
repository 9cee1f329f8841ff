"""Index arithmetic of the in-place product for any layout, replayed on the host (no GPU).

``tests/host_replay/replay_any.cpp`` is compiled with g++ under AddressSanitizer
and UndefinedBehaviorSanitizer with the planner and the index functions the
kernel uses (``csrc/any_index.hpp``).  It rebuilds every tile's LDS image load by
load on random contractions (odd sizes, K tails, K-major and complex operands,
16- and 4-byte loads) and checks bounds, alignment and that every MFMA operand
read finds the element the offset tables name.
"""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2007_08056_amd", "csrc")
ROCM_INCLUDE = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")


@pytest.mark.timeout(600)
def test_any_layout_product_replay(tmp_path):
    gxx = shutil.which(os.environ.get("CXX", "g++"))
    if gxx is None or not os.path.isdir(ROCM_INCLUDE):
        pytest.skip("needs g++ and the ROCm headers")
    exe = str(tmp_path / "replay_any")
    build = [gxx, "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-I", ROCM_INCLUDE,
             "-I", os.path.join(ROOT, "include"), "-I", CSRC,
             "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-fno-omit-frame-pointer",
             os.path.join(ROOT, "tests", "host_replay", "replay_any.cpp"), os.path.join(CSRC, "plan.cpp"), "-o", exe]
    r = subprocess.run(build, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout + r.stderr
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:halt_on_error=1",
               UBSAN_OPTIONS="print_stacktrace=1:halt_on_error=1")
    r = subprocess.run([exe, "400"], capture_output=True, text=True, timeout=500, env=env)
    print(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr[-4000:]
    assert " 0 failures" in r.stdout
    m = re.search(r"A along K (\d+), K-major (\d+), pairs (\d+); complex V in place (\d+); 4-byte only (\d+); "
                  r"split-bf16 (\d+)\), (\d+) K-step tails", r.stdout)
    assert m and all(int(x) > 0 for x in m.groups()), r.stdout
    m = re.search(r"(\d+) direct subgroup plans \((\d+) clear W\)", r.stdout)
    assert m and int(m.group(1)) > int(m.group(2)) > 0, r.stdout
