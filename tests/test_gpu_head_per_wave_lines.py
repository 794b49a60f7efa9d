"""Where token-major calls change from the head-major mapping to a wave per KV head: on both sides of the lower lines, by the kernel
that ran and against the fp64 oracle; and calls in the groups of heads that fused steps with more than eight KV heads take (which
groups those are, on both sides of every line, tests/host/host_calls.cpp reads from the launches)."""
import numpy as np
import pytest
import torch

import workloads
from oracle import spd_oracle as orc
from test_gpu_parity import DEV, TOL, _check_one, _oracle_outputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2409_19134_amd as spd
    c = spd.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def _lens(users, steps):
    """Uneven lengths that make `steps` 32-token steps, last steps partly filled."""
    share = np.full(users, steps // users)
    share[0] += steps - share.sum()
    shift = min(int(share[-1]) // 3, 20)
    for u in range(0, users - 1, 2):
        share[u] += shift
        share[u + 1] -= shift
    return [int(32 * s - (7 * u) % 32) for u, s in enumerate(share)]


def _run(ctx, d, Hkv, G, users, head_steps, fused, want_hpw, below=0, dtype=torch.bfloat16, paged=False):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    steps = -(-head_steps * cus // Hkv) - below
    lo = [1 + 9 * u % 60 for u in range(users)]
    lp = _lens(users, steps - sum(-(-n // 32) for n in lo) if fused else steps)
    wl = workloads.random_case(411, dtype, users, Hkv * G, Hkv, d, lp, lo, device=DEV, layout="nhd", paged=paged)
    step, _ = _check_one(ctx, wl, _oracle_outputs(orc.from_workload(wl), None), None, TOL[dtype], fused)
    if not fused:
        ctx.spd_partial_attn_private(step.shape, wl.q, step.private, step.a_in, step.lse_in)
        torch.cuda.synchronize()
    name = ctx.spd_last_kernel_name()
    assert name.startswith("partial_mfma_kernel<"), name
    assert (name.split(", ")[4] == "true") == want_hpw, name


@pytest.mark.parametrize("d,Hkv,G,users,line,fused", [
    (64, 8, 4, 10, 40, True), (64, 8, 8, 12, 40, True), (64, 32, 1, 4, 40, True), (64, 8, 3, 11, 32, False), (64, 16, 2, 7, 32, False),
    (128, 8, 4, 16, 41, False), (128, 32, 1, 4, 41, False)])
@pytest.mark.parametrize("below", [0, 1])
def test_lines(ctx, d, Hkv, G, users, line, fused, below):
    _run(ctx, d, Hkv, G, users, line, fused, below == 0, below)


@pytest.mark.parametrize("d,Hkv,G,users,line,fused", [(64, 8, 4, 10, 40, True), (64, 16, 2, 7, 32, False), (128, 8, 4, 16, 41, False)])
@pytest.mark.parametrize("below", [0, 1])
def test_lines_in_pages_of_fp16(ctx, d, Hkv, G, users, line, fused, below):
    _run(ctx, d, Hkv, G, users, line, fused, below == 0, below, dtype=torch.float16, paged="token_major")


@pytest.mark.parametrize("d,Hkv,G,users,head_steps,fused", [
    (64, 8, 4, 9, 45, True),       # 72 rows: their pieces are too many
    (64, 4, 4, 24, 28, True),      # fewer than eight heads
    (128, 8, 4, 16, 45, True),     # a fused step of 128-value heads: from 65
    (128, 8, 8, 16, 45, False)])   # eight query heads per KV head
def test_calls_that_stay_head_major(ctx, d, Hkv, G, users, head_steps, fused):
    _run(ctx, d, Hkv, G, users, head_steps, fused, False)


@pytest.mark.parametrize("d,Hkv,G,users,dtype,paged", [
    (128, 12, 1, 9, torch.bfloat16, False), (64, 20, 2, 5, torch.float16, "token_major"), (128, 32, 1, 3, torch.float16, False),
    (64, 16, 5, 1, torch.bfloat16, False)])
def test_fused_steps_in_groups_of_four(ctx, d, Hkv, G, users, dtype, paged):
    """(The kernel's name shows the mapping, not the group.)"""
    _run(ctx, d, Hkv, G, users, 66, True, True, dtype=dtype, paged=paged)


@pytest.mark.parametrize("d,users,lp,lo,fused", [(64, 12, 3200, 160, True), (64, 12, 2720, 0, False), (128, 16, 4096, 32, True)])
def test_capture_of_a_view_that_has_grown_across_a_line(d, users, lp, lo, fused):
    """Eight heads on 256 units: run eagerly below the line, captured 64 tokens later above it - on the schedules of before."""
    import paper_2409_19134_amd as spd
    own = spd.Context(0)
    grow = 64
    wl = workloads.random_case(412, torch.bfloat16, users, 32, 8, d, [lp + (0 if fused else grow)] * users, [lo + grow] * users, device=DEV,
                               layout="nhd")
    side_of = "public" if fused else "private"
    full = getattr(wl, side_of).lens.copy()
    side = torch.cuda.Stream()

    def call(step):
        if fused:
            step.run_fused(wl.q)
        else:
            own.spd_partial_attn_private(step.shape, wl.q, step.private, step.a_in, step.lse_in)

    with torch.cuda.stream(side):
        getattr(wl, side_of).lens = (full - grow).astype(np.int32)
        call(spd.DecodeStep.from_workload(own, wl))
        torch.cuda.synchronize()
        before, builds = own.spd_last_kernel_name(), own.spd_get_schedule_stats()[0]
        getattr(wl, side_of).lens = full
        step = spd.DecodeStep.from_workload(own, wl)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            call(step)
        assert own.spd_last_kernel_name() == before and before.split(", ")[4] == "false"
        hw = orc.from_workload(wl)
        A, _, _ = orc.partial(hw, hw.public if fused else hw.private)
        got = step.a_out if fused else step.a_in
        for _ in range(3):
            got.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert np.abs(got.cpu().double().numpy().reshape(A.shape) - A).max() <= TOL[wl.dtype]
        assert own.spd_get_schedule_stats()[0] == builds
        call(step)                                     # outside a capture the rule decides
        torch.cuda.synchronize()
        assert own.spd_last_kernel_name().split(", ")[4] == "true"
    own.close()
