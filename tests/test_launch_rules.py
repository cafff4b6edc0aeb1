"""The rules that size a launch (csrc/host_logic.h), built with g++ under
AddressSanitizer and UndefinedBehaviorSanitizer (tests/host/
test_launch_rules.cpp).  No GPU."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1611_03226_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_launch_rules_under_sanitizers(tmp_path):
    exe = str(tmp_path / "launch_rules")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
           f"-I{CSRC}", os.path.join(HERE, "host", "test_launch_rules.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120,
                       env=dict(os.environ, ASAN_OPTIONS="verify_asan_link_order=0"))
    assert r.returncode == 0 and "launch rules: ok" in r.stdout, r.stdout + r.stderr
