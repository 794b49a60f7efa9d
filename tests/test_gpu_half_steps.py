"""The streaming kernel's forms for long pieces and for fp32 rows read through buffer descriptors: 16-bit rows in 16-token steps
(-128 channels of dtypes 1 and 2 in the kernel's name), fp32 on 4x4 matrix blocks (of 3).  Against the fp64 oracle at lengths around their tiles, in the storage
modes and with the append; the tolerances are the parity tests' (sums of the same values in another order)."""
import copy

import numpy as np
import pytest
import torch

import workloads
from oracle import spd_oracle as orc
from test_gpu_append import _clone_side, _set_last_token
from test_gpu_parity import DEV, TOL, _check_one, _oracle_outputs, maxerr

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2409_19134_amd as spd
    c = spd.Context(0)
    c.spd_set_option(spd.SPD_OPT_TARGET_WG_PER_CU, 1)      # long pieces from small inputs: with 32 KV heads 8 per head on 256 units
    yield c
    torch.cuda.synchronize()
    c.close()


def _ran(ctx, code):
    """code: the kernel's dtype, "+" behind it for the dtype's other form."""
    name = ctx.spd_last_kernel_name()
    assert name.startswith(f"partial_mfma_kernel<{code[0]}, {-128 if code.endswith('+') else 128}, "), name


def _nan_behind(side):
    """What lies behind a user's last token in its head-major buffer is never part of a result."""
    for u, n in enumerate(side.lens):
        for t in (side.k[u], side.v[u]):
            t[:, int(n):] = float("nan")


# private tokens: 12 and more 32-token steps a piece, ends around a 16-token tile and around one step of all four waves (64)
LENS = [([3072], [0]), ([4081], [1]), ([4095], [15]), ([4096], [16]), ([4097], [17]), ([4127], [33]), ([4161], [65]), ([2063, 2064], [64, 129]),
        ([9, 5000], [0, 31])]


@pytest.mark.parametrize("lp,lo", LENS)
@pytest.mark.parametrize("dtype,code,G,storage", [
    (torch.bfloat16, "1+", 1, "hnd"), (torch.bfloat16, "1+", 4, "hnd_exact"), (torch.bfloat16, "1+", 16, "paged"),
    (torch.float16, "2+", 3, "hnd"), (torch.float16, "2+", 2, "paged"), (torch.float32, "3+", 4, "hnd"), (torch.float32, "3+", 1, "hnd_exact"),
    (torch.float32, "3", 2, "paged")])
def test_forms_at_tile_edges(ctx, lp, lo, dtype, code, G, storage):
    Hkv = 32
    wl = workloads.random_case(311, dtype, len(lp), Hkv * G, Hkv, 128, lp, lo, device=DEV, layout="hnd" if storage == "paged" else storage,
                               paged=storage == "paged")
    hw = orc.from_workload(wl)
    want = _oracle_outputs(hw, None)
    if storage == "hnd":
        _nan_behind(wl.private)
        _nan_behind(wl.public)
    _check_one(ctx, wl, want, None, TOL[dtype], True)
    _ran(ctx, code)


@pytest.mark.parametrize("lo", [[1, 16], [17, 15], [700, 32]])
@pytest.mark.parametrize("dtype,code,storage", [(torch.bfloat16, "1+", "hnd"), (torch.float16, "2+", "paged"), (torch.float32, "3", "hnd")])
def test_append(ctx, lo, dtype, code, storage):
    import paper_2409_19134_amd as spd
    Hkv, U = 32, 2
    wl = workloads.random_case(312, dtype, U, Hkv * 4, Hkv, 128, [3000, 1100], lo, device=DEV, layout="hnd", paged=storage == "paged")
    g = torch.Generator(device=DEV).manual_seed(979)
    k_new, v_new = (torch.randn((U, Hkv, 128), generator=g, device=DEV).to(dtype) for _ in range(2))
    want = copy.copy(wl)
    want.public = _clone_side(wl.public)
    for u in range(U):
        _set_last_token(want.public, u, k_new[u], v_new[u])
    step = spd.DecodeStep.from_workload(ctx, wl)
    step.run_fused(wl.q, k_new=k_new, v_new=v_new)
    torch.cuda.synchronize()
    _ran(ctx, code)
    Y, _ = orc.attention(orc.from_workload(want))
    assert maxerr(step.y, Y) <= TOL[dtype]
    for a, b in zip((wl.public.k_pool, wl.public.v_pool) if storage == "paged" else (*wl.public.k, *wl.public.v),
                    (want.public.k_pool, want.public.v_pool) if storage == "paged" else (*want.public.k, *want.public.v)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("n,page,code", [(12288, 16, "1+"), (12544, 16, "1"), (12544, 0, "1+")])
def test_long_pieces_of_one_owner(ctx, n, page, code):
    """48 and 49 steps a piece: pages leave the 16-token form there, contiguous rows do not."""
    wl = workloads.random_case(313, torch.bfloat16, 1, 32, 32, 128, [n], [5], device=DEV, layout="hnd", paged=bool(page))
    step, _ = _check_one(ctx, wl, _oracle_outputs(orc.from_workload(wl), None), None, TOL[wl.dtype], False)
    ctx.spd_partial_attn_private(step.shape, wl.q, step.private, step.a_in, step.lse_in)
    torch.cuda.synchronize()
    _ran(ctx, code)


def test_strides_past_the_descriptors_range():
    """Tokens 2^27 bytes apart (fp32: 128 MB): the 64-bit form takes what does not lie end to end."""
    import paper_2409_19134_amd as spd
    own = spd.Context(0)
    n, d, stride = 5, 128, 1 << 25
    K, V = (torch.empty((n - 1) * stride + d, device=DEV) for _ in range(2))
    rows = [torch.randn((n, d), device=DEV, generator=torch.Generator(device=DEV).manual_seed(s)) for s in (1, 2)]
    for t in range(n):
        K[t * stride:t * stride + d], V[t * stride:t * stride + d] = rows[0][t], rows[1][t]
    q = torch.randn((1, 2, d), device=DEV, generator=torch.Generator(device=DEV).manual_seed(3))
    own.spd_set_option(spd.SPD_OPT_HEAD_PER_WAVE, 0)       # the split kernels
    out, lse = own.spd_partial_attn_private(spd.make_shape(torch.float32, 2, 1, d, 0.1), q, spd.KVView([n], stride, 0, k=[K], v=[V]))
    assert own.spd_last_kernel_name().startswith("partial_mfma_kernel<3, 128, "), own.spd_last_kernel_name()
    s = (q[0].double() @ rows[0].double().t()) * 0.1
    assert (out[0].double() - torch.softmax(s, 1) @ rows[1].double()).abs().max().item() <= TOL[torch.float32]
    assert (lse[0].double() - torch.logsumexp(s, 1)).abs().max().item() <= TOL[torch.float32]
    own.close()


@pytest.mark.parametrize("n", [1, 17, 33, 81])
@pytest.mark.parametrize("Hkv,stride", [(1, 132), (3, 3 * 128), (1, 128)])
def test_nothing_behind_a_row_is_read(n, Hkv, stride):
    """fp32 rows, one token into a tile, whose rest is there and holds NaN: tokens end to end are read through descriptors, those
    between which the token stride leaves room are not."""
    import paper_2409_19134_amd as spd
    own = spd.Context(0)
    own.spd_set_option(spd.SPD_OPT_HEAD_PER_WAVE, 0)       # the split kernels
    d, whole = 128, -(-n // 16) * 16
    g = torch.Generator(device=DEV).manual_seed(n)
    K, V = (torch.full((whole, stride), float("nan"), device=DEV) for _ in range(2))
    rows = [torch.randn((n, Hkv, d), device=DEV, generator=g) for _ in range(2)]
    for t, r in zip((K, V), rows):
        t[:n, :Hkv * d] = r.view(n, Hkv * d)
    q = torch.randn((1, 2 * Hkv, d), device=DEV, generator=g)
    out, lse = own.spd_partial_attn_private(spd.make_shape(torch.float32, 2 * Hkv, Hkv, d, 0.1), q, spd.KVView([n], stride, d, k=[K], v=[V]))
    assert own.spd_last_kernel_name().startswith(f"partial_mfma_kernel<3, {-128 if stride == d else 128}, "), own.spd_last_kernel_name()
    k, v = (r.double().transpose(0, 1) for r in rows)
    s = torch.stack([q[0, 2 * h:2 * h + 2].double() @ k[h].t() for h in range(Hkv)]) * 0.1
    want = torch.stack([torch.softmax(s[h], 1) @ v[h] for h in range(Hkv)])
    assert (out.view(Hkv, 2, d).double() - want).abs().max().item() <= TOL[torch.float32]
    assert (lse.view(Hkv, 2).double() - torch.logsumexp(s, 2)).abs().max().item() <= TOL[torch.float32]
    own.close()
