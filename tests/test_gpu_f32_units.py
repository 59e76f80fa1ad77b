"""The fp32 half-step units (operands as three bf16 planes) at the edges of
their tiles: 1 to 128 rows a block, head dimensions that fill and do not fill
the 64-, 96- and 128-wide tiles, on full and ragged sequences, pre-padded and
with per-sequence lengths, against the fp64 oracle at the fp32 bar."""
import numpy as np
import pytest

import oracle
import parity
import synth_inputs as si

pytestmark = pytest.mark.gpu

TOL = 1e-5


@pytest.fixture(scope="module")
def ma():
    import torch

    assert torch.cuda.is_available(), "no GPU visible"
    import paper_2505_18698_amd as lib

    return lib


@pytest.mark.parametrize("n,m,b,d,T", [
    (16 * 16, 16, 16, 64, 2), (17 * 33 - 5, 17, 33, 96, 2), (64 * 64, 64, 64, 128, 2), (65 * 16, 65, 16, 64, 3),
    (128 * 128 - 7, 128, 128, 64, 2), (1, 1, 1, 4, 2), (31 * 5, 31, 5, 100, 1), (5 * 127, 5, 127, 60, 2),
    (9 * 20 - 3, 9, 20, 88, 2), (16 * 12, 16, 12, 128, 3),
])
def test_units(ma, n, m, b, d, T):
    import torch

    B, H = 2, 1
    q, k, v = si.random_qkv(B, H, n, d, "f32", seed=6, scale=1.5)
    tq, tk, tv = (torch.from_numpy(x).cuda() for x in (q, k, v))
    lens = np.array([n, max(1, n // 3)], dtype=np.int32)

    out = ma.monarch_attn_fwd(tq, tk, tv, torch.full_like(tq, float("nan")), m, b, T).double().cpu().numpy()
    ref = oracle.monarch_attention(q, k, v, m, b, T)
    assert oracle.rel_frobenius(out, ref) <= TOL
    assert parity.worst_class(out, ref, b)[0] <= parity.class_bar(TOL)

    flip = [torch.flip(x, (2,)).contiguous() for x in (tq, tk, tv)]
    pre = ma.monarch_attn_fwd_prepad(*flip, torch.full_like(tq, float("nan")), m, b, T)
    assert np.array_equal(torch.flip(pre, (2,)).double().cpu().numpy(), out)  # the same problem, row-reversed

    var = ma.monarch_attn_fwd_varlen(tq, tk, tv, torch.full_like(tq, float("nan")), torch.from_numpy(lens).cuda(), m, b, T)
    var = var.double().cpu().numpy()
    ref = oracle.monarch_attention_varlen(q, k, v, lens, m, b, T)
    assert np.isfinite(var).all() and oracle.rel_frobenius(var, ref) <= TOL


@pytest.mark.parametrize("m,b,d", [(9, 20, 64), (16, 12, 96), (2, 63, 128)])
def test_workgroups_that_take_several_units(ma, m, b, d):
    """More units than the device holds at once (12 waves a compute unit at
    most): every head's bits are those of a call on that head alone."""
    import torch

    H, n = 400, m * b - 1
    q, k, v = (torch.randn(1, H, n, d, device="cuda") for _ in range(3))
    out = ma.monarch_attn_fwd(q, k, v, torch.full_like(q, float("nan")), m, b, 2)
    for h in (0, 201, H - 1):
        one = [x[:, h:h + 1].contiguous() for x in (q, k, v)]
        alone = ma.monarch_attn_fwd(*one, torch.full_like(one[0], float("nan")), m, b, 2)
        assert torch.equal(alone[0, 0], out[0, h])
