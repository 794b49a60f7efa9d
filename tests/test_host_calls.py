"""The built library's host side without a GPU: launches and uploads recorded by a stand-in HIP runtime (see
tests/host/host_calls.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_uploads_and_launches_on_a_recorded_runtime(tmp_path):
    """What the calls ask of the runtime: the static step's schedules stay inside their parts of the fixed array."""
    exe = str(tmp_path / "host_calls")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-rdynamic", "-o", exe, os.path.join(ROOT, "tests", "host", "host_calls.cpp"), "-ldl"]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout[-3000:]
    lib = os.path.join(ROOT, "paper_2409_19134_amd", "libspd_hip.so")
    run = subprocess.run([exe, lib], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert run.returncode == 0 and run.stdout.strip().endswith("ok"), run.stdout[-3000:]
