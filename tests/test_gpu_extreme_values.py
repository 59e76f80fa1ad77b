"""Values at the end of fp32's range and infinities, where operands are held as
bf16 planes: a finite value of any size is a finite operand, and an infinite V
or dO gives what fp32 products give, an infinite column of O or dV, and leaves
the rest as it is.  Against the fp64 oracle, column by column (one column is
some 1e38 times the others), at the bars of the other parity tests."""
import numpy as np
import pytest

import oracle
import oracle.backward as ob
import synth_inputs as si
from test_gpu_backward import TOL, _td, gpu_grads, ma  # noqa: F401

pytestmark = pytest.mark.gpu

MAX = {"f32": np.float32(3.4028234663852886e38), "bf16": np.float32(3.3895313892515355e38), "f16": np.float32(65504.0)}
SHAPES = [(5, 7, 64, 1), (5, 7, 64, 2), (20, 33, 72, 2), (64, 64, 128, 2), (128, 128, 48, 1)]  # m, b, d, T
COL = 5


def inputs(m, b, d, dtype):
    n = m * b - 1
    q, k, v = si.random_qkv(1, 1, n, d, dtype, seed=11, scale=0.5)  # every weight well above zero
    return n, q, k, v, si.random_cotangent((1, 1, n, d), dtype, seed=11)


def column_errors(x, ref):
    return np.linalg.norm(x - ref, axis=-2) / np.linalg.norm(ref, axis=-2)


def forward(ma, dtype, q, k, v, m, b, T):  # noqa: F811
    import torch

    tq, tk, tv = (torch.from_numpy(x).to(_td(dtype)).cuda() for x in (q, k, v))
    return ma.monarch_attn_fwd(tq, tk, tv, torch.full_like(tq, float("nan")), m, b, T).double().cpu().numpy()


@pytest.mark.parametrize("m,b,d,T", SHAPES)
@pytest.mark.parametrize("sign", [1, -1])
def test_fp32_forward_v(ma, m, b, d, T, sign):  # noqa: F811
    n, q, k, v, _ = inputs(m, b, d, "f32")
    v[0, 0, n // 3, COL] = sign * MAX["f32"]
    out = forward(ma, "f32", q, k, v, m, b, T)
    assert np.isfinite(out).all()
    assert column_errors(out, oracle.monarch_attention(q, k, v, m, b, T)).max() <= 1e-5

    v[0, 0, n // 3, COL] = sign * np.inf
    inf = forward(ma, "f32", q, k, v, m, b, T)
    assert (inf[..., COL] == sign * np.inf).all()
    rest = np.arange(d) != COL
    assert np.array_equal(inf[..., rest], out[..., rest])


@pytest.mark.parametrize("m,b,d,T", SHAPES)
@pytest.mark.parametrize("sign", [1, -1])
def test_fp32_forward_k(ma, m, b, d, T, sign):  # noqa: F811
    """In a column that the queries leave out, a key at the end of the range
    changes nothing.  (Beyond 3.396e38, where bf16 rounds to infinity, but off
    the last value: alpha_L's products sum e K with weights e up to 1 before
    they are divided by the sum of e.)"""
    n, q, k, v, _ = inputs(m, b, d, "f32")
    q[..., COL] = 0
    k[0, 0, n // 3, COL] = np.float32(sign * 3.4e38)
    out = forward(ma, "f32", q, k, v, m, b, T)
    assert np.isfinite(out).all()
    assert oracle.rel_frobenius(out, oracle.monarch_attention(q, k, v, m, b, T)) <= 1e-5


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("m,b,d,T", SHAPES)
@pytest.mark.parametrize("sign", [1, -1])
def test_gradient_infinite_dout(ma, dtype, m, b, d, T, sign):  # noqa: F811
    n, q, k, v, g = inputs(m, b, d, dtype)
    plain = gpu_grads(ma, q, k, v, g, m, b, T, dtype)
    row = n // 3
    g[0, 0, row, COL] = sign * np.inf
    dq, dk, dv = gpu_grads(ma, q, k, v, g, m, b, T, dtype)
    rest, classes = np.arange(d) != COL, np.arange(n) % b != row % b
    assert (dv[..., COL] == sign * np.inf).all()
    assert np.array_equal(dv[..., rest], plain[2][..., rest])
    # the pull-back of the softmax makes NaN of it (inf - inf): the row's residue class of dq, and all keys
    assert np.array_equal(dq[:, :, classes], plain[0][:, :, classes])
    assert not np.isfinite(dq[:, :, row]).any() and not np.isfinite(dk).any()


@pytest.mark.parametrize("m,b,d,T", SHAPES)
def test_gradient_large_v(ma, m, b, d, T):  # noqa: F811
    """V at the end of the range: dV does not depend on V, and dQ and dK are finite."""
    n, q, k, v, g = inputs(m, b, d, "f32")
    plain = gpu_grads(ma, q, k, v, g, m, b, T, "f32")
    g[..., COL] *= np.float32(2.0 ** -20)
    v[0, 0, n // 3, COL] = MAX["f32"]
    got = gpu_grads(ma, q, k, v, g, m, b, T, "f32")
    ref = ob.autograd_grads(q[0, 0], k[0, 0], v[0, 0], g[0, 0], m, b, T)
    rest = np.arange(d) != COL
    assert np.array_equal(got[2][..., rest], plain[2][..., rest])
    for name, x, r in zip(("dq", "dk", "dv"), got, ref):
        assert np.isfinite(x).all(), name
        assert oracle.rel_frobenius(x[0, 0], r) <= TOL["f32"], name


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("m,b,d,T", SHAPES)
@pytest.mark.parametrize("down", [0, 4])
def test_gradient_large_dout(ma, dtype, m, b, d, T, down):  # noqa: F811
    """dO at the end of the range (times 2^-down): the sums over a row of the
    factors' gradients, not yet divided by the sum of the weights, do not overflow."""
    n, q, k, v, g = inputs(m, b, d, dtype)
    plain = gpu_grads(ma, q, k, v, g, m, b, T, dtype)
    row = n // 3
    v *= np.float32(0.25)  # <dO, Y> within the range
    g[0, 0, row, COL] = MAX[dtype] * np.float32(2.0 ** -down)
    got = gpu_grads(ma, q, k, v, g, m, b, T, dtype)
    ref = ob.autograd_grads(q[0, 0], k[0, 0], v[0, 0], g[0, 0], m, b, T)
    rest = np.arange(d) != COL
    assert np.array_equal(got[2][..., rest], plain[2][..., rest])
    for name, x, r in zip(("dq", "dk", "dv"), got, ref):
        assert np.isfinite(x).all(), name
        assert oracle.rel_frobenius(x[0, 0], r) <= TOL[dtype], name
