"""The gradient's units at the edges of their tiles and LDS plans: 16- to
128-row tiles of both updates, head dimensions that fill and do not fill the
64-, 96- and 128-wide tiles, and the three element types (1, 2 and 3 planes),
against the fp64 autograd oracle with the bars of test_gpu_backward.
"""
import numpy as np
import pytest

import oracle.backward as ob
import parity
import synth_inputs as si
from test_gpu_backward import TOL, _td, gpu_grads, ma, run_case  # noqa: F401

pytestmark = pytest.mark.gpu

# n, m, b, d, T
SHAPES = {
    "bf16": [(256, 16, 16, 64, 2), (17 * 33, 17, 33, 96, 2), (64 * 65, 64, 65, 64, 2), (65 * 64 - 3, 65, 64, 128, 1),
             (128 * 128, 128, 128, 128, 2), (127 * 128 - 1, 127, 128, 88, 2), (16 * 128, 16, 128, 8, 3)],
    "f16": [(15 * 16 - 7, 15, 16, 128, 3), (32 * 32, 32, 32, 64, 2), (128 * 100, 128, 100, 96, 2),
            (128 * 128 - 5, 128, 128, 128, 2), (40 * 64, 40, 64, 64, 1)],
    "f32": [(16 * 16, 16, 16, 128, 2), (33 * 31 - 2, 33, 31, 96, 2), (64 * 64, 64, 64, 128, 2),
            (128 * 120 - 9, 128, 120, 64, 2), (128 * 16, 128, 16, 4, 1)],
}


@pytest.mark.parametrize("dtype,shape", [(t, s) for t in SHAPES for s in SHAPES[t]])
def test_unit_tiles(ma, dtype, shape):  # noqa: F811
    n, m, b, d, T = shape
    heads = 1 if n > 4096 else 2
    run_case(ma, 1, heads, n, m, b, d, T, dtype, seed=5)


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("m,b,d", [(8, 48, 64), (20, 12, 64), (100, 70, 32)])
def test_blocks_of_padding_only(ma, dtype, m, b, d):  # noqa: F811
    """Two steps with whole key blocks of padding: c_R of such a block is zero,
    and its reciprocal must not reach the gradient."""
    import torch

    lens = np.array([m * b, 2 * b + 1, 1], dtype=np.int32)
    B, n, T = len(lens), m * b, 2
    q, k, v = si.random_qkv(B, 1, n, d, dtype, seed=8, scale=1.5)
    g = si.random_cotangent((B, 1, n, d), dtype, seed=8)
    tq, tk, tv, tg = (torch.from_numpy(x).to(_td(dtype)).cuda() for x in (q, k, v, g))
    outs = [torch.full_like(tq, float("nan")) for _ in range(3)]
    ma.monarch_attn_bwd_varlen(tq, tk, tv, tg, *outs, torch.from_numpy(lens).cuda(), m, b, T)
    for i, r in enumerate(lens):
        ref = ob.autograd_grads(q[i, 0, :r], k[i, 0, :r], v[i, 0, :r], g[i, 0, :r], m, b, T, batch_padding=True)
        for name, x, y in zip(("dq", "dk", "dv"), outs, ref):
            x = x[i, 0].double().cpu().numpy()
            assert np.isfinite(x).all() and (x[r:] == 0).all(), (name, i)
            err = np.linalg.norm(x[:r] - y) / max(np.linalg.norm(y), 1e-30)
            # one real row: its only key has weight 1, so dq and dk are zero up to rounding
            assert err <= parity.class_bar(TOL[dtype]) or np.linalg.norm(x[:r] - y) <= 1e-5, (name, i, err)


@pytest.mark.parametrize("shift", [-60, 60])
def test_gradient_is_linear_in_dout(ma, shift):  # noqa: F811
    """Scaling dout by a power of two scales every product of the sweep, plane
    by plane, without rounding: the fp32 gradients scale bit for bit (inputs of
    scale 0.5 give logits of a few units, so that no weight, and no product
    with one, comes near the underflow threshold)."""
    m, b, d, T = 40, 33, 64, 2
    n = m * b - 4
    q, k, v = si.random_qkv(1, 1, n, d, "f32", seed=9, scale=0.5)
    g = si.random_cotangent((1, 1, n, d), "f32", seed=9)
    one = gpu_grads(ma, q, k, v, g, m, b, T, "f32")
    two = gpu_grads(ma, q, k, v, np.ldexp(g, shift).astype(np.float32), m, b, T, "f32")
    for name, x, y in zip(("dq", "dk", "dv"), one, two):
        assert np.array_equal(np.ldexp(x, shift), y), name
