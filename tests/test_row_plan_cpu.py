"""CPU tests of the host plans that the block operator and the HEX08 owner
kernel run (tests/sanitize/row_check.cpp), under AddressSanitizer and
UndefinedBehaviorSanitizer, and under ThreadSanitizer (host code only)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2107_11541_amd", "csrc")
SANITIZERS = {"memory": ["-fsanitize=address,undefined", "-fno-sanitize-recover=undefined"], "threads": ["-fsanitize=thread"]}


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
@pytest.mark.parametrize("which", list(SANITIZERS))
def test_row_and_owner_plans(tmp_path, which):
    exe = str(tmp_path / "row_check")
    r = subprocess.run(["g++", "-std=c++17", "-pthread", "-O2", "-g", "-fno-omit-frame-pointer", *SANITIZERS[which],
                        "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "sanitize", "row_check.cpp"),
                        os.path.join(CSRC, "plan.cpp"), os.path.join(CSRC, "rowplan.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0", UBSAN_OPTIONS="print_stacktrace=1")
    env.pop("LD_PRELOAD", None)
    p = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=600)
    assert p.returncode == 0 and "0 failed checks" in p.stdout, (p.stdout[-2000:], p.stderr[-6000:])
