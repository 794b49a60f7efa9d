"""Calls of short rows run on the whole-rows kernel: one launch, one workgroup per (user, KV head), no closing kernel.
Against the oracle and against the split kernels, which the options that shape or pick them still select."""
import numpy as np
import pytest
import torch

import workloads
from test_gpu_parity import TOL, _check_one, _oracle_outputs, run_step
from oracle import spd_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
OUTPUTS = ("a_in", "lse_in", "a_out", "lse_out", "y", "lse", "w_in")


@pytest.fixture(scope="module")
def ctx():
    import paper_2409_19134_amd as spd
    c = spd.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


@pytest.fixture(scope="module")
def split_ctx():
    """A context whose calls all take the split schedule (an option that picks its kernels is set)."""
    import paper_2409_19134_amd as spd
    c = spd.Context(0)
    c.spd_set_option(spd.SPD_OPT_STEPS_IN_FLIGHT, 1)
    yield c
    torch.cuda.synchronize()
    c.close()


def _both_ways(ctx, split_ctx, wl):
    """Every call form on whole rows against the oracle, and the fused step against the split kernels."""
    want = _oracle_outputs(orc.from_workload(wl), None)
    for fused in (False, True, "two_parties"):
        step, _ = _check_one(ctx, wl, want, None, None, fused)
        assert ctx.spd_last_kernel_name().startswith("whole_rows_kernel<"), ctx.spd_last_kernel_name()
    ref = run_step(split_ctx, wl, True)
    assert not split_ctx.spd_last_kernel_name().startswith("whole_rows")
    for name in OUTPUTS:
        a, b = getattr(step, name), getattr(ref, name)
        fin = torch.isfinite(b)
        assert torch.equal(fin, torch.isfinite(a)), name
        # both are within TOL of the same value
        assert (a[fin] - b[fin]).abs().max().item() <= 2 * TOL[wl.dtype] if fin.any() else True, name


# lengths around a step (32 tokens; 16 for 512-byte rows), and totals around twelve of them: 1, 11, 12, 13 and more steps,
# with one owner empty, both, and the owners' border inside a wave's share
PRIVATE = [0, 1, 31, 32, 33, 320, 352, 384, 385, 0, 100, 190, 17]
PUBLIC = [0, 0, 1, 33, 31, 64, 32, 0, 1, 385, 97, 193, 400]


@pytest.mark.parametrize("dtype,d,Hq,Hkv", [(torch.bfloat16, 128, 8, 2), (torch.bfloat16, 128, 32, 2), (torch.float16, 64, 3, 3),
                                            (torch.float16, 128, 14, 2), (torch.float32, 64, 4, 1), (torch.float32, 64, 5, 1),
                                            (torch.float32, 128, 4, 2), (torch.float32, 128, 16, 1),
                                            (torch.bfloat16, 128, 22, 2), (torch.float16, 128, 13, 1), (torch.float32, 128, 15, 1)])
@pytest.mark.parametrize("storage", ["hnd", "nhd", "hnd_exact", "paged", "paged_tm"])
def test_step_and_wave_edges(ctx, split_ctx, dtype, d, Hq, Hkv, storage):
    paged = {"paged": True, "paged_tm": "token_major"}.get(storage, False)
    div = 2 if dtype == torch.float32 and d == 128 else 1           # the same number of steps
    wl = workloads.random_case(501, dtype, len(PRIVATE), Hq, Hkv, d, [-(-x // div) for x in PRIVATE], [-(-x // div) for x in PUBLIC],
                               device=DEV, layout="nhd" if paged else storage, paged=paged)
    _both_ways(ctx, split_ctx, wl)


# (The rule takes a few users' rows whole up to 14 steps above the share, a fused step, or 16, one owner's call: the lengths of
# the tests below with few users stay under that.)
# 256 compute units: a workgroup each (up to 12 waves), up to two rows per unit (8 waves, or 4 for rows of up to 16 steps),
# more rows than are resident at once (4 waves, launched by length)
@pytest.mark.parametrize("U,top", [(1, 430), (31, 700), (33, 400), (60, 700), (65, 300), (300, 200)])
def test_workgroup_sizes_and_launch_order(ctx, split_ctx, U, top):
    rng = np.random.default_rng(U)
    lo = rng.integers(0, 90, U)
    wl = workloads.random_case(502, torch.bfloat16, U, 16, 8, 64 if U == 300 else 128, rng.integers(top - 150, top, U).tolist(),
                               lo.tolist(), device=DEV, layout="hnd")
    _both_ways(ctx, split_ctx, wl)


def test_one_owners_nan_stays_out_of_the_others_partial(ctx):
    wl = workloads.random_case(503, torch.bfloat16, 3, 8, 2, 128, [250, 40, 90], [180, 70, 33], device=DEV, layout="hnd")
    clean = run_step(ctx, wl, True)
    keep = {name: getattr(clean, name).clone() for name in OUTPUTS}
    wl.private.v[1][0, 5, :] = float("nan")              # user 1, KV head 0, token 5
    step = run_step(ctx, wl, True)
    assert ctx.spd_last_kernel_name().startswith("whole_rows_kernel<")
    rows = slice(0, 4)                                    # the query heads of KV head 0
    assert torch.isnan(step.a_in[1, rows]).all() and torch.isnan(step.y[1, rows]).all()
    assert torch.equal(step.a_out, keep["a_out"]) and torch.equal(step.lse_out, keep["lse_out"])
    for name in ("a_in", "y"):
        a, b = getattr(step, name).clone(), keep[name].clone()
        a[1, rows] = b[1, rows] = 0
        assert torch.equal(a, b), name


@pytest.mark.parametrize("split", [False, True])
@pytest.mark.parametrize("Hq,Hkv,d", [(4, 1, 64), (10, 2, 128), (32, 2, 64)])
def test_an_infinite_value_stays_infinite(ctx, split_ctx, split, Hq, Hkv, d):
    """fp32 caches whose V holds an infinity: the channel's partials are that infinity, all others are finite, also where the
    infinity is in the last chunk (split) or the last wave's share (whole rows), which is read in place of absent ones."""
    c = split_ctx if split else ctx
    lp, lo = ([300, 520, 140, 33], [150, 277, 260, 140]) if split else ([100, 110, 120, 33], [70, 66, 61, 110])
    for at in (0, 1, 2):                                    # in the first, a middle and the last token but one
        wl = workloads.random_case(507, torch.float32, 4, Hq, Hkv, d, lp, lo, device=DEV, layout="hnd")
        for u, (side, n) in enumerate(((wl.private, lp[0]), (wl.public, lo[1]), (wl.private, lp[2]), (wl.public, lo[3]))):
            side.v[u][Hkv - 1, (0, n // 2, n - 2)[at], 5 + u] = float("inf") if u % 2 else -float("inf")
        step = run_step(c, wl, True)
        assert c.spd_last_kernel_name().startswith("whole_rows") != split
        G = Hq // Hkv
        for u in range(4):
            inf = torch.zeros((Hq, d), dtype=torch.bool, device=DEV)
            inf[Hq - G:, 5 + u] = True
            mine, other = (step.a_out, step.a_in) if u % 2 else (step.a_in, step.a_out)
            for t in (mine[u], step.y[u]):
                assert torch.equal(t == (float("inf") if u % 2 else -float("inf")), inf), (at, u)
                assert torch.isfinite(t[~inf]).all(), (at, u)
            assert torch.isfinite(other[u]).all()


@pytest.mark.parametrize("steps", [1, 2, 3, 4])
@pytest.mark.parametrize("dtype,Hq,Hkv,d", [(torch.bfloat16, 4, 1, 64), (torch.float16, 2, 2, 128), (torch.bfloat16, 24, 3, 128),
                                            (torch.float32, 5, 1, 64), (torch.float32, 3, 1, 128)])
def test_up_to_four_waves(ctx, split_ctx, dtype, Hq, Hkv, d, steps):
    """Workgroups of up to four waves combine both owners' slots at once: every border of the owners among up to four steps, a step
    shared by no wave, one owner empty, a thread per channel and four channels a thread; and an infinite V value, which the last slot
    holds, stays the only one (it stands in, with weight 0, for absent slots)."""
    step = 16 if dtype == torch.float32 and d == 128 else 32
    pairs = [(i, j) for i in range(steps + 1) for j in range(steps + 1 - i)]
    lp, lo = [i * step - (7 if i else 0) for i, _ in pairs], [j * step for _, j in pairs]
    wl = workloads.random_case(508, dtype, len(pairs), Hq, Hkv, d, lp, lo, device=DEV, layout="hnd")
    _both_ways(ctx, split_ctx, wl)
    if dtype != torch.float32:  # (16-bit probabilities are pairs, whose low part may be 0)
        return
    for u, (a, b) in enumerate(zip(lp, lo)):
        if a + b:  # the last step's first token (the last one stands in, with weight 0, for a ragged step's absent tokens)
            (wl.public.v[u][0, b - step] if b else wl.private.v[u][0, (a - 1) // step * step])[u] = float("inf")
    out = run_step(ctx, wl, True)
    assert ctx.spd_last_kernel_name().startswith("whole_rows")
    for u, (a, b) in enumerate(zip(lp, lo)):
        inf = torch.zeros((Hq, d), dtype=torch.bool, device=DEV)
        inf[:Hq // Hkv, u] = a + b > 0
        mine, other = (out.a_out, out.a_in) if b else (out.a_in, out.a_out)
        for t in (mine[u], out.y[u]):
            assert torch.equal(t == float("inf"), inf) and torch.isfinite(t[~inf]).all(), u
        assert torch.isfinite(other[u]).all(), u


@pytest.mark.parametrize("dtype,Hq,Hkv,U,top,paged,append,three", [
    (torch.float32, 8, 2, 210, 700, False, False, True),      # up to two rows a unit: eight waves each, one at a time
    (torch.float32, 10, 2, 210, 700, True, False, True),
    (torch.float16, 4, 2, 210, 1200, True, False, True),
    (torch.bfloat16, 4, 2, 210, 1200, False, True, True),
    (torch.bfloat16, 4, 2, 210, 1200, True, True, False),     # the append in pages keeps two at a time
    (torch.bfloat16, 4, 2, 210, 1200, False, False, False),   # (an instance of which a unit holds one anyway)
    (torch.float32, 3, 3, 300, 120, False, False, True),      # four waves each, 900 rows
    (torch.float32, 10, 2, 600, 90, False, False, True),      # 1200 rows
    (torch.float16, 4, 2, 600, 90, True, False, False)])
def test_forms_for_rows_that_wait_for_others(ctx, split_ctx, dtype, Hq, Hkv, U, top, paged, append, three):
    """64-channel rows, more than are resident at once: the form held to three waves per SIMD takes the calls that its rule says, with
    the results of the split kernels; the other calls keep the plain instance."""
    import paper_2409_19134_amd as spd
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256
    rng = np.random.default_rng(U + top)
    wl = workloads.random_case(509, dtype, U, Hq, Hkv, 64, rng.integers(top // 3, top, U).tolist(), rng.integers(1, 60, U).tolist(),
                               device=DEV, layout="hnd", paged=paged)
    gen = torch.Generator(device=DEV).manual_seed(510)
    new = [torch.randn((U, Hkv, 64), generator=gen, device=DEV).to(dtype) for _ in range(2)] if append else [None, None]
    out = []
    for c in (ctx, split_ctx):
        step = spd.DecodeStep.from_workload(c, wl)
        for name in OUTPUTS:
            getattr(step, name).fill_(float("nan"))
        step.run_fused(wl.q, None, *new)        # (the second call writes the same rows to the cache again)
        torch.cuda.synchronize()
        out.append(step)
    name = ctx.spd_last_kernel_name()
    assert name.startswith("whole_rows_kernel<") and (name.split(", ")[1] == "-64") == three, name
    for key in OUTPUTS:
        a, b = getattr(out[0], key), getattr(out[1], key)
        assert torch.isfinite(a).all() and (a - b).abs().max().item() <= 2 * TOL[dtype], key   # both are within TOL of the same value
    if not append:
        _check_one(ctx, wl, _oracle_outputs(orc.from_workload(wl), None), None, None, True)


@pytest.mark.parametrize("paged", [False, True])
def test_decode_loop_appends_on_whole_rows(ctx, paged):
    """Twenty steps of a growing public cache: the appended rows reach the cache, the schedule is found again, results
    agree with the oracle on the cache as it then is."""
    import paper_2409_19134_amd as spd
    U, Hkv, d, steps = 4, 2, 128, 20
    lo0 = np.array([1, 31, 60, 128])
    wl = workloads.random_case(504, torch.bfloat16, U, 8, Hkv, d, [200, 33, 64, 1], (lo0 + steps).tolist(), device=DEV, layout="hnd",
                               paged=paged)
    full_lens = wl.public.lens
    gen = torch.Generator(device=DEV).manual_seed(505)
    own = spd.Context(0)
    for i in range(steps):
        wl.public.lens = (lo0 + i + 1).astype(np.int32)
        new = [torch.randn((U, Hkv, d), generator=gen, device=DEV).to(torch.bfloat16) for _ in range(2)]
        step = spd.DecodeStep.from_workload(own, wl)
        step.run_fused(wl.q, None, *new)
        torch.cuda.synchronize()
        assert own.spd_last_kernel_name().startswith("whole_rows_kernel<")
        Y, _ = orc.attention(orc.from_workload(wl))      # the oracle reads the cache the call has written
        assert np.abs(step.y.cpu().double().numpy().reshape(Y.shape) - Y).max() <= TOL[wl.dtype]
        for u in range(U):
            t = int(wl.public.lens[u]) - 1
            for side, row in zip((wl.public.k_pool if paged else wl.public.k[u], wl.public.v_pool if paged else wl.public.v[u]), new):
                at = side[int(wl.public.block_table[u, t // 16]), :, t % 16] if paged else side[:, t]
                assert torch.equal(at, row[u])
    builds, hits = own.spd_get_schedule_stats()
    assert builds == 2 and hits == 2 * (steps - 1)
    wl.public.lens = full_lens
    own.close()


@pytest.mark.parametrize("entry", ["fused", "public", "merge"])
def test_capture_of_a_view_that_has_grown_across_the_rule(entry):
    """A schedule serves a view whose lengths have grown by up to 64 tokens, also while the stream is captured: so it does
    where the growth takes the rows from whole to split - the remembered way of taking them is kept and nothing is built."""
    import paper_2409_19134_amd as spd
    U = 4
    lp, lo = ([400, 100, 97, 128], [64] * U) if entry == "fused" else ([64] * U, [560, 100, 97, 128])
    wl = workloads.random_case(506, torch.bfloat16, U, 8, 2, 128, lp, lo, device=DEV, layout="hnd")
    lens = wl.public.lens.copy()
    own = spd.Context(0)
    side = torch.cuda.Stream()

    def call(step):
        if entry == "fused":
            step.run_fused(wl.q)
        elif entry == "public":
            own.spd_partial_attn_public_batched(step.shape, wl.q, step.public, step.a_out, step.lse_out)
        else:
            own.spd_public_attn_merge(step.shape, wl.q, step.public, step.a_in, step.lse_in, step.a_out, step.lse_out, step.y,
                                      step.lse, step.w_in)

    def step_at(grown):
        wl.public.lens = (lens - 60 + grown).astype(np.int32)
        return spd.DecodeStep.from_workload(own, wl)

    seen = set()
    with torch.cuda.stream(side):
        first = step_at(0)
        for t in (first.a_in, first.lse_in):
            t.zero_()
        call(first)
        torch.cuda.synchronize()
        builds = own.spd_get_schedule_stats()[0]
        for grown in (5, 30, 60):
            step = step_at(grown)
            for t in (step.a_in, step.lse_in):
                t.zero_()
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=side):
                call(step)
            seen.add(own.spd_last_kernel_name().split("<")[0])
            for _ in range(3):
                step.a_out.fill_(float("nan"))
                graph.replay()
                torch.cuda.synchronize()
                A, _, _ = orc.partial(orc.from_workload(wl), orc.from_workload(wl).public)
                assert np.abs(step.a_out.cpu().double().numpy().reshape(A.shape) - A).max() <= TOL[wl.dtype]
        assert own.spd_get_schedule_stats()[0] == builds
        assert seen == {"whole_rows_kernel"}
        call(step_at(60))                          # outside a capture the rule decides: these rows are split
        torch.cuda.synchronize()
        assert own.spd_last_kernel_name().startswith("partial_mfma_kernel")
    own.close()
