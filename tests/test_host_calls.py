"""The built library's host side without a GPU: launches and uploads recorded by a stand-in HIP runtime (see
tests/host/host_calls.cpp)."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_uploads_and_launches_on_a_recorded_runtime(tmp_path, resource_report):
    """What the calls ask of the runtime: the static step's schedules stay inside their parts of the fixed array and are those of
    the ordinary step where they fit, a whole-rows launch inside 64 KB of LDS; calls beside a capture of another stream; what a
    captured step counts as found and builds; on both sides of their lines the mapping rule with its head groups, the half steps
    and the descriptors; the last instance's template arguments."""
    static_lds = {int(x) for name, x in re.findall(r"Function Name: (\S+)(?:(?!Function Name).)*?LDS Size \[bytes/block\]: (\d+)",
                                                   resource_report, re.S) if "whole_rows_kernel" in name}
    assert len(static_lds) == 1, static_lds
    exe = str(tmp_path / "host_calls")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-rdynamic", "-o", exe, os.path.join(ROOT, "tests", "host", "host_calls.cpp"), "-ldl"]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout[-3000:]
    lib = os.path.join(ROOT, "paper_2409_19134_amd", "libspd_hip.so")
    run = subprocess.run([exe, lib, str(static_lds.pop())], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert run.returncode == 0 and run.stdout.strip().endswith("ok"), run.stdout[-3000:]
