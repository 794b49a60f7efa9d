"""spd_decode_step_static (the decode step on the library's fixed scratch array, for callers that cannot allocate)
against spd_decode_step: same inputs, every output bit for bit, on two calls in a row, the second one smaller."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
OUTPUTS = ("a_in", "lse_in", "a_out", "lse_out", "y", "lse", "w_in")


def _both(ctx, wl, k_new=None, v_new=None):
    """(outputs of spd_decode_step, outputs of spd_decode_step_static) for one workload."""
    import paper_2409_19134_amd as spd
    got = []
    for static in (False, True):
        step = spd.DecodeStep.from_workload(ctx, wl)
        for name in OUTPUTS:
            getattr(step, name).fill_(float("nan"))
        fn = ctx.spd_decode_step_static if static else ctx.spd_decode_step
        fn(step.shape, wl.q, step.private, step.public, step.a_in, step.lse_in, step.a_out, step.lse_out, step.y,
           step.lse, step.w_in, None, k_new, v_new)
        torch.cuda.synchronize()
        got.append({name: getattr(step, name).clone() for name in OUTPUTS})
    return got


def _same(a, b):
    for name in OUTPUTS:
        assert not torch.isnan(b[name]).any(), name
        assert torch.equal(a[name].view(torch.int32), b[name].view(torch.int32)), name


def test_static_step_equals_decode_step_twice_second_smaller():
    import paper_2409_19134_amd as spd
    ctx = spd.Context(0)
    big = workloads.make_workload(2, DEV)                       # the headline workload: 16 users, ~38 000 tokens
    small = workloads.random_case(77, torch.bfloat16, 3, 32, 8, 128, [700, 0, 33], [17, 64, 0], device=DEV)
    for wl in (big, small, big):
        ref, got = _both(ctx, wl)
        _same(ref, got)
    ctx.close()


def test_static_step_other_storage_modes_and_append():
    import paper_2409_19134_amd as spd
    ctx = spd.Context(0)
    paged = workloads.make_workload(5, DEV, len_div=64, n_users=6)
    f32 = workloads.make_workload(1, DEV)
    token_major = workloads.make_workload(4, DEV, len_div=8, n_users=40, layout="nhd")
    for wl in (paged, f32, token_major):
        ref, got = _both(ctx, wl)
        _same(ref, got)
    wl = workloads.random_case(78, torch.bfloat16, 4, 32, 8, 128, [3000, 100, 900, 64], [300, 900, 5, 1], device=DEV)
    gen = torch.Generator(device=DEV).manual_seed(79)
    k_new = torch.randn((4, 8, 128), generator=gen, device=DEV).to(torch.bfloat16)
    v_new = torch.randn((4, 8, 128), generator=gen, device=DEV).to(torch.bfloat16)
    ref, got = _both(ctx, wl, k_new, v_new)
    _same(ref, got)
    ctx.close()


def test_static_step_refuses_what_does_not_fit():
    """A schedule of more work items than the array has room for: an error before anything is launched."""
    import paper_2409_19134_amd as spd
    ctx = spd.Context(0)
    U = 2100                                     # 2100 users x 8 KV heads x 2 pieces x 48 bytes > 512 KiB
    lens = np.full(U, 40, dtype=np.int32)
    wl = workloads.random_case(80, torch.bfloat16, U, 32, 8, 128, lens, lens, device=DEV)
    step = spd.DecodeStep.from_workload(ctx, wl)
    step.y.fill_(7.0)
    with pytest.raises(spd.binding.SpdError) as e:
        ctx.spd_decode_step_static(step.shape, wl.q, step.private, step.public, step.a_in, step.lse_in, step.a_out,
                                   step.lse_out, step.y, step.lse, step.w_in)
    assert e.value.code == spd.binding.SPD_ERR_WORKSPACE
    torch.cuda.synchronize()
    assert float(step.y.min()) == 7.0 == float(step.y.max())       # nothing ran
    step.run_fused(wl.q)                                           # the allocating entry point takes the same step
    torch.cuda.synchronize()
    assert not torch.isnan(step.y).any()
    ctx.close()


def test_static_step_in_a_hip_graph_without_warm_up():
    """Recorded into a graph as the very first call on its view (schedules travel in kernel arguments), replayed with
    fresh queries between other eager work."""
    import paper_2409_19134_amd as spd
    ctx = spd.Context(0)
    wl = workloads.random_case(81, torch.bfloat16, 5, 32, 8, 128, [2000, 100, 0, 900, 64], [300, 900, 5, 0, 1], device=DEV)
    other = workloads.random_case(82, torch.bfloat16, 2, 32, 8, 128, [500, 90], [30, 9], device=DEV)
    step = spd.DecodeStep.from_workload(ctx, wl)
    q = wl.q.clone()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        ctx.spd_decode_step_static(step.shape, q, step.private, step.public, step.a_in, step.lse_in, step.a_out,
                                   step.lse_out, step.y, step.lse, step.w_in, torch.cuda.current_stream())
    gen = torch.Generator(device=DEV).manual_seed(83)
    for rep in range(3):
        q.copy_(torch.randn(q.shape, generator=gen, device=DEV).to(q.dtype))
        torch.cuda.synchronize()
        ref_step = spd.DecodeStep.from_workload(ctx, wl)
        ref_step.run_fused(q)
        # eager work of another view on the same array between the replays
        o = spd.DecodeStep.from_workload(ctx, other)
        ctx.spd_decode_step_static(o.shape, other.q, o.private, o.public, o.a_in, o.lse_in, o.a_out, o.lse_out, o.y, o.lse,
                                   o.w_in)
        torch.cuda.synchronize()
        step.y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for name in OUTPUTS:
            assert torch.equal(getattr(step, name).view(torch.int32), getattr(ref_step, name).view(torch.int32)), (rep, name)
    ctx.close()


def test_static_step_whose_whole_rows_tables_exceed_the_array():
    """Token-major, 2500 users of short rows: the split schedule has an item per four heads and fits, the tables of rows
    taken whole have one per head and do not - the step takes the split schedule."""
    import paper_2409_19134_amd as spd
    ctx = spd.Context(0)
    wl = workloads.random_case(84, torch.bfloat16, 2500, 8, 8, 64, [64] * 2500, [32] * 2500, device=DEV, layout="nhd")
    step = spd.DecodeStep.from_workload(ctx, wl)
    step.run_fused(wl.q)
    assert ctx.spd_last_kernel_name().startswith("whole_rows_kernel<")     # the allocating step has the room
    ctx.spd_decode_step_static(step.shape, wl.q, step.private, step.public, step.a_in, step.lse_in, step.a_out,
                               step.lse_out, step.y, step.lse, step.w_in)
    assert ctx.spd_last_kernel_name().startswith("partial_mfma_kernel<")
    torch.cuda.synchronize()
    split = spd.Context(0)
    split.spd_set_option(spd.SPD_OPT_STEPS_IN_FLIGHT, 2)                   # what the head-per-wave mapping takes anyway
    ref = spd.DecodeStep.from_workload(split, wl)
    ref.run_fused(wl.q)
    torch.cuda.synchronize()
    _same({n: getattr(ref, n) for n in OUTPUTS}, {n: getattr(step, n) for n in OUTPUTS})
    split.close()
    ctx.close()


@pytest.mark.parametrize("users,Hq,Hkv,d,lp,lo", [(12, 32, 8, 64, 3400, 200), (9, 12, 12, 128, 5000, 300), (6, 16, 16, 128, 9000, 300)])
def test_static_step_takes_the_fused_steps_mapping(users, Hq, Hkv, d, lp, lo):
    """Token-major views between the mapping rule's lines: 64-channel heads from 40 head steps per unit, groups of four of more
    than eight KV heads."""
    import paper_2409_19134_amd as spd
    ctx = spd.Context(0)
    wl = workloads.random_case(85, torch.bfloat16, users, Hq, Hkv, d, [lp - 31 * u for u in range(users)], [lo] * users, device=DEV,
                               layout="nhd")
    ref, got = _both(ctx, wl)
    assert ctx.spd_last_kernel_name().split(", ")[4] == "true"             # head per wave
    _same(ref, got)
    ctx.close()


def test_static_step_with_a_split_of_its_own_where_the_fused_steps_does_not_fit():
    """16 query heads per KV head of 64 channels: the partials of a wave per head are more than the array holds."""
    import paper_2409_19134_amd as spd
    from oracle import spd_oracle as orc
    ctx = spd.Context(0)
    wl = workloads.random_case(86, torch.bfloat16, 12, 128, 8, 64, [3400 - 31 * u for u in range(12)], [200] * 12, device=DEV, layout="nhd")
    ref, got = _both(ctx, wl)
    assert ctx.spd_last_kernel_name().split(", ")[4] == "false"            # head-major
    Y, _ = orc.attention(orc.from_workload(wl))
    for out in (ref, got):
        assert np.abs(out["y"].cpu().double().numpy().reshape(Y.shape) - Y).max() <= 2e-3
    ctx.close()
