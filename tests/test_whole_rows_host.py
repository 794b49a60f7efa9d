"""The whole-rows tables and the rule that picks them, on the host (see tests/host/whole_rows_fuzz.cpp)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not found")
def test_whole_rows_tables_and_rule_under_asan_ubsan(tmp_path):
    """Random views in every storage mode: the rows' addresses are the split schedule's, every token is covered, the
    launch order is a permutation by length; the rule's wave counts and limits; the kernel's division by the wave count."""
    exe = str(tmp_path / "whole_rows_fuzz")
    cmd = [HIPCC, "--offload-arch=gfx950", "-O1", "-g", "-std=c++17", "-x", "hip",
           "-Xarch_host", "-fsanitize=address,undefined", "-Xarch_host", "-fno-sanitize-recover=undefined",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-o", exe, os.path.join(ROOT, "tests", "host", "whole_rows_fuzz.cpp")]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout[-3000:]
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=0", UBSAN_OPTIONS="print_stacktrace=1")
    run = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, env=env, timeout=300)
    assert run.returncode == 0 and run.stdout.strip().endswith("ok 600"), run.stdout[-3000:]
