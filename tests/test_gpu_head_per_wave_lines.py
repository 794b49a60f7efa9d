"""Where token-major calls change from the head-major mapping to a wave per KV head, and the head groups that fused steps with more
than eight KV heads take: on both sides of each line, by the kernel that ran and against the fp64 oracle."""
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
    _run(ctx, d, Hkv, G, users, 66, True, True, dtype=dtype, paged=paged)
