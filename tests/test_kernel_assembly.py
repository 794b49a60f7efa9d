"""What the compiler makes of the kernels, read from the assembly of this library's own sources (no GPU needed)."""
import importlib.util
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not found")
    spec = importlib.util.spec_from_file_location("spd_build", os.path.join(ROOT, "paper_2409_19134_amd", "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    out = str(tmp_path_factory.mktemp("assembly") / "kernels.s")
    cmd = [HIPCC, *(f for f in build.HIPCC_FLAGS if f != "-shared"), "--cuda-device-only", "-S", "-o", out,
           os.path.join(ROOT, "paper_2409_19134_amd", "csrc", "spd_api.hip")]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout[-3000:]
    with open(out) as f:
        return f.read()


def test_all_of_a_buffer_loads_offset_is_range_checked(assembly):
    """Rows end inside a tile, and what lies behind them is kept out by the descriptor's range: the offset's scalar part, which
    the range check is not specified to cover, is zero in every load through a descriptor."""
    loads = re.findall(r"^\s+(buffer_load_\w+ .*)$", assembly, re.M)
    assert len(loads) >= 30, len(loads)
    scalar = [l for l in loads if not re.match(r"buffer_load_\w+ v\[\d+:\d+\], v\d+, s\[\d+:\d+\], 0 offen( |$)", l)]
    assert not scalar, (len(scalar), scalar[:4])


def test_what_a_workgroup_needs_first_is_preloaded(assembly):
    """The streaming, whole-rows and closing kernels ask for their item or row with their first instructions: the parameters that this
    takes (RowsHead's 14 dwords, PartialHead's 13, CloseHead's 7) arrive in scalar registers."""
    least = {"partial_mfma_kernel": 13, "whole_rows_kernel": 14, "close_kernel": 7}
    seen = dict.fromkeys(least, 0)
    for name, n in re.findall(r"\.amdhsa_kernel (\S+)(?:(?!\.end_amdhsa_kernel).)*?preload_length (\d+)", assembly, re.S):
        for kernel, dwords in least.items():
            if kernel in name:
                assert int(n) >= dwords, (name, n)
                seen[kernel] += 1
    assert all(seen.values()), seen
