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
    """The parameters from which the streaming, whole-rows and closing kernels find their item or row (PartialHead's and RowsHead's 14
    dwords, CloseHead's 8) arrive in scalar registers."""
    least = {"partial_mfma_kernel": 14, "whole_rows_kernel": 14, "close_kernel": 8}
    seen = dict.fromkeys(least, 0)
    for name, n in re.findall(r"\.amdhsa_kernel (\S+)(?:(?!\.end_amdhsa_kernel).)*?preload_length (\d+)", assembly, re.S):
        for kernel, dwords in least.items():
            if kernel in name:
                assert int(n) >= dwords, (name, n)
                seen[kernel] += 1
    assert all(seen.values()), seen


def _until_asked(body, load):
    """A kernel's instructions from its entry to the load that the pattern names.  Of the whole-rows kernel the path without a launch
    order (its first branch taken, on a comparison of the order with null); the code in front of the entry, for firmware that does not
    preload, is left out."""
    lines = body.split(".p2align\t8", 1)[1].splitlines()[2:]  # (behind the alignment: the entry's label)
    skip_to, seen = None, []
    for line, following in zip(lines, lines[1:]):
        op = line.split(";")[0].strip()
        if skip_to:
            skip_to = None if op == skip_to + ":" else skip_to
            continue
        seen.append(op)
        if re.match(load, op):
            return seen
        branch = re.match(r"\s+s_cbranch_scc1 (\S+)", following)
        if branch and re.match(r"s_cmp_eq_u64 \S+, 0$", op):
            skip_to = branch.group(1)
    raise AssertionError(f"no {load}")


@pytest.mark.parametrize("kernel,load", [("partial_mfma_kernel", r"s_load_dwordx8 \S+ \S+ 0x10$"),  # dwords 4 to 11 of the item
                                         ("whole_rows_kernel", r"s_load_dwordx8 \S+ \S+ 0x0$"),     # the row
                                         ("close_kernel", r"global_load_dwordx2 ")])                 # the row's chunks
def test_a_workgroup_asks_for_its_item_before_it_waits(assembly, kernel, load):
    """Nothing is waited for in front of the load of a workgroup's item or row (whole rows: without a launch order): a trip to the
    arguments there is what preloading is for."""
    bodies = re.findall(rf"^(_Z\S*{kernel}\S*):.*?\n(.*?)^\.Lfunc_end", assembly, re.S | re.M)
    assert len(bodies) >= 32, len(bodies)
    for name, body in bodies:
        asked = _until_asked(body, load)
        assert not [op for op in asked if op.startswith("s_waitcnt")], (name, asked)


def _metadata(assembly, kernel):
    """(demangled template arguments, metadata block) of every instance of a kernel."""
    for block in re.findall(r"^  - \.agpr_count:.*?(?=^  - \.agpr_count:|^amdhsa\.target)", assembly, re.S | re.M):
        name = re.search(r"\.name:\s+(\S+)", block).group(1)
        if kernel in name:
            yield tuple(int(v.replace("n", "-")) for v in re.findall(r"L[ib](n?\d+)E", name)), block


@pytest.mark.parametrize("kernel", ["partial_mfma_kernel", "whole_rows_kernel"])
def test_the_arguments_lie_where_the_kernel_reads_them(assembly, kernel):
    """Both kernels read their last parameter, the owners' arguments, at an offset from the argument segment that the size of the head in
    front gives: 56 bytes.  There it is, 240 bytes (two owners' 120, or whole rows' 8 + 5 pairs of 16, 72 of results and two
    owners' 40 of pages), and nothing but the runtime's hidden arguments behind it."""
    count = 0
    for args, block in _metadata(assembly, kernel):
        explicit = [(int(at), int(size)) for at, size, kind in
                    re.findall(r"- \.offset:\s+(\d+)\s+\.size:\s+(\d+)\s+\.value_kind:\s+(\w+)", block) if not kind.startswith("hidden")]
        assert explicit == [(0, 32), (32, 16), (48, 8), (56, 240)], (args, explicit)
        count += 1
    assert count >= 32


def test_short_rows_of_64_channels_keep_four_waves_per_simd(assembly):
    """Many short rows are bound by the workgroups that a compute unit holds: with at most 128 vector registers a fourth wave fits a SIMD.
    These instances are at most that large: fp32 (16x16 blocks) without the append, 16-bit rows in pages without it, contiguous with it.
    The form for rows that a unit gets one after the other (64 channels, negative) is larger, so that it gets one at a time."""
    at_most_128 = {(0, 64, 0, 0), (0, 64, 1, 0), (1, 64, 1, 0), (2, 64, 1, 0), (1, 64, 0, 1), (2, 64, 0, 1)}
    seen = {args: int(re.search(r"\.vgpr_count:\s+(\d+)", block).group(1)) for args, block in _metadata(assembly, "whole_rows_kernel")}
    forms = {args for args in seen if args[1] < 0}
    assert len(seen) == 40 and at_most_128 <= set(seen) and len(forms) == 8, sorted(seen)
    assert all(seen[args] <= 128 for args in at_most_128), {args: seen[args] for args in at_most_128}
    assert all(128 < seen[args] <= 168 for args in forms), {args: seen[args] for args in forms}
    # (a form where the plain instance would hold two such rows a unit, and for the append in pages, which gains by two, none)
    assert forms == {(t, -64, p, a) for t, c, p, a in seen if c == 64 and seen[t, c, p, a] <= 128 and not (p and a)}, sorted(forms)


def test_short_rows_in_pages_spill_no_scalar_register(assembly):
    """A row's launch is latency: what a paged run needs of its owner is read where the run begins, not held (and spilled, an instruction
    each way and a wait in front of the row) beside the other owner's."""
    spills = {args: int(re.search(r"\.sgpr_spill_count:\s+(\d+)", block).group(1)) for args, block in _metadata(assembly, "whole_rows_kernel")}
    paged = {args: n for args, n in spills.items() if args[2]}
    assert len(paged) == 20 and not any(paged.values()), paged
