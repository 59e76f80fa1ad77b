"""The one-workgroup-per-head kernel at every tile width (d up to 128): the
automatic path gives the bits of the half-steps, on full and ragged heads,
padded batches, pre-padding and with the objective, for fewer heads than the
device holds at once and for more (a workgroup then takes several)."""
import numpy as np
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ma():
    import torch

    assert torch.cuda.is_available(), "no GPU visible"
    import paper_2505_18698_amd as lib

    return lib


def both(ma, call):
    out = []
    for path in (ma.PATH_HALF_STEPS, ma.PATH_AUTO):
        prev = ma.monarch_attn_set_path(path)
        try:
            out.append(call())
        finally:
            ma.monarch_attn_set_path(prev)
    return out


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("B,H,n,m,b,d,T", [
    (1, 2, 256, 16, 16, 72, 3), (1, 3, 1, 1, 1, 128, 1), (2, 2, 15 * 14 - 13, 15, 14, 96, 2), (1, 2, 16, 1, 16, 104, 2),
    (1, 2, 16, 16, 1, 80, 4), (3, 200, 9 * 7, 9, 7, 64, 2), (2, 280, 16 * 5 - 4, 16, 5, 128, 2), (1, 2, 40, 5, 8, 8, 2),
])
def test_bits_of_the_half_steps(ma, dtype, B, H, n, m, b, d, T):
    import torch

    td = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    q, k, v = (torch.from_numpy(x).to(td).cuda() for x in si.random_qkv(B, H, n, d, dtype, seed=3, scale=1.5)[:3])
    lens = torch.from_numpy(si.sequence_lengths(B, n, seed=4)).cuda()
    lens[-1] = 0

    def plain():
        return ma.monarch_attn_fwd(q, k, v, torch.full_like(q, float("nan")), m, b, T)

    def prepad():
        return ma.monarch_attn_fwd_prepad(q, k, v, torch.full_like(q, float("nan")), m, b, T)

    def varlen():
        return ma.monarch_attn_fwd_varlen(q, k, v, torch.full_like(q, float("nan")), lens, m, b, T)

    def objective():
        obj = torch.full((B, H, T), float("nan"), device="cuda")
        out, obj = ma.monarch_attn_fwd_objective(q, k, v, torch.full_like(q, float("nan")), obj, m, b, T)
        return torch.cat((out.float().flatten(), obj.flatten()))

    for call in (plain, prepad, varlen, objective):
        one, two = both(ma, call)
        torch.cuda.synchronize()
        assert torch.isfinite(one.float()).all(), call.__name__
        assert torch.equal(one, two), call.__name__


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("B,H,n,m,b,d,T", [
    (3, 100, 15 * 14 - 13, 15, 14, 64, 3), (3, 100, 16 * 16, 16, 16, 72, 2), (3, 100, 9 * 7 - 2, 9, 7, 128, 2),
    (2, 300, 4 * 16, 4, 16, 64, 2), (1, 2, 16 * 5 - 4, 16, 5, 96, 4),
])
def test_gradient_recompute_gives_the_bits_of_the_half_steps(ma, dtype, B, H, n, m, b, d, T):
    """The states that the recompute keeps, of every step and for several heads
    a workgroup: the same gradients as from the half-steps' states."""
    import torch

    td = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    q, k, v = (torch.from_numpy(x).to(td).cuda() for x in si.random_qkv(B, H, n, d, dtype, seed=5, scale=1.5)[:3])
    g = torch.from_numpy(si.random_cotangent((B, H, n, d), dtype, seed=5)).to(td).cuda()
    lens = torch.from_numpy(si.sequence_lengths(B, n, seed=6)).cuda()
    lens[-1] = 0
    ma.monarch_attn_timing_enable(True)
    try:
        for varlen in (False, True):
            def call():
                out = [torch.full_like(q, float("nan")) for _ in range(3)]
                if varlen:
                    ma.monarch_attn_bwd_varlen(q, k, v, g, *out, lens, m, b, T)
                else:
                    ma.monarch_attn_bwd(q, k, v, g, *out, m, b, T)
                return torch.stack(out), [kind for kind, _ in ma.monarch_attn_timing_read()]

            (one, kinds), (two, auto) = both(ma, call)
            assert kinds[:2 * T - 1] == ["r_half_step", "l_half_step"] * (T - 1) + ["r_half_step_final"]
            assert auto[0] == "monarch_fused_head" and auto[1:] == kinds[2 * T - 1:]
            assert torch.isfinite(one.float()).all() and torch.equal(one, two), varlen
    finally:
        ma.monarch_attn_timing_enable(False)


@pytest.mark.parametrize("B,H,m,b,d,T,forward,recompute", [
    (1, 23, 16, 16, 128, 1, False, False), (1, 24, 16, 16, 128, 1, True, False), (1, 4, 15, 14, 104, 1, False, False),
    (1, 11, 16, 16, 96, 1, False, False), (1, 12, 16, 16, 72, 1, True, False), (1, 4, 15, 14, 96, 1, True, False),
    (1, 4, 8, 8, 128, 1, True, False), (3, 300, 16, 16, 64, 1, True, False), (1, 2, 16, 16, 64, 2, True, True),
    (1, 63, 16, 16, 128, 2, True, False), (2, 32, 16, 16, 128, 2, True, True), (1, 2, 4, 16, 96, 2, True, True),
    (1, 1, 16, 16, 128, 3, True, True), (1, 63, 8, 15, 128, 2, True, True), (1, 63, 8, 16, 104, 2, True, False),
    (1, 4, 16, 16, 96, 2, True, False), (1, 4, 16, 15, 72, 2, True, True),
    # many tiny heads (256 compute units)
    (1, 256, 1, 1, 72, 1, True, False), (1, 257, 4, 5, 72, 1, False, False), (1, 512, 4, 6, 72, 1, True, False),
    (1, 1025, 4, 8, 128, 1, False, False), (2, 2000, 8, 8, 128, 1, True, False), (1, 1024, 2, 5, 104, 2, True, False),
    (1, 1025, 2, 5, 104, 2, False, False), (1, 512, 1, 1, 72, 2, True, False), (1, 1028, 1, 4, 72, 3, False, False),
    (4, 900, 2, 5, 72, 3, False, False), (4, 1000, 4, 4, 72, 3, True, False), (1, 512, 4, 6, 64, 2, True, True),
    (1, 513, 4, 6, 64, 2, True, False), (2, 1500, 8, 8, 96, 2, True, True), (1, 512, 1, 1, 96, 3, True, True),
    (1, 1025, 4, 4, 96, 3, True, False), (1, 256, 1, 1, 64, 2, True, True),
])
def test_one_launch_where_it_is_faster(ma, B, H, m, b, d, T, forward, recompute):
    """The lines of the automatic path: one step of few large heads, many tiny
    heads, and the recompute of one step, run on the half-steps."""
    import torch

    half = ["r_half_step", "l_half_step"] * (T - 1) + ["r_half_step_final"]
    q, k, v, g = (torch.randn(B, H, m * b, d, device="cuda", dtype=torch.bfloat16) for _ in range(4))
    out, grads = torch.empty_like(q), [torch.empty_like(q) for _ in range(3)]
    ma.monarch_attn_timing_enable(True)
    try:
        ma.monarch_attn_fwd(q, k, v, out, m, b, T)
        assert [kind for kind, _ in ma.monarch_attn_timing_read()] == (
            ["monarch_fused_head"] if forward else half + ["monarch_apply"])
        lens = torch.full((B,), m * b, device="cuda", dtype=torch.int32)
        ma.monarch_attn_fwd_varlen(q, k, v, out, lens, m, b, T)
        few = T == 1 and d > 96 and m * b >= 64 and B * H < 24  # with lengths, heads of 64 rows up
        assert [kind for kind, _ in ma.monarch_attn_timing_read()] == (
            ["monarch_fused_head"] if forward and not few else half + ["monarch_apply"])
        ma.monarch_attn_bwd(q, k, v, g, *grads, m, b, T)
        kinds = [kind for kind, _ in ma.monarch_attn_timing_read()]
        assert kinds == (["monarch_fused_head"] if recompute else half) + ["l_bwd", "r_bwd"] * T
    finally:
        ma.monarch_attn_timing_enable(False)


def test_what_wide_small_heads_need_is_unchanged(ma):
    """d > 64: forcing the one-workgroup-per-head path stays refused, and the
    no-allocation call keeps its scratch limit."""
    import torch

    q = torch.zeros(1, 700, 256, 72, device="cuda", dtype=torch.bfloat16)
    out = torch.empty_like(q)
    prev = ma.monarch_attn_set_path(ma.PATH_FUSED)
    try:
        with pytest.raises(ma.MonarchAttnError):
            ma.monarch_attn_fwd(q, q, q, out, 16, 16, 1)
    finally:
        ma.monarch_attn_set_path(prev)
    assert ma.monarch_attn_workspace_bytes(1, 700, 256, 72, 16, 16, 1, ma.MA_BF16) > ma.NOALLOC_SCRATCH_BYTES
    with pytest.raises(ma.MonarchAttnError):
        ma.monarch_attn_fwd_noalloc(q, q, q, out, 16, 16, 1)
    half = q[:, :300].contiguous()
    ma.monarch_attn_fwd_noalloc(half, half, half, torch.empty_like(half), 16, 16, 1)
