"""The binding's argument checks (no GPU): on every entry point that takes
tensors, each one that is no device tensor, not contiguous or not of q's
shape, dtype and device is refused by name before the library is called."""
import pytest
import torch

import paper_2505_18698_amd as ma


@pytest.mark.parametrize("call", [
    lambda x: ma.monarch_attn_fwd(x, x, x, x, 2, 2, 1),
    lambda x: ma.monarch_attn_fwd_noalloc(x, x, x, x, 2, 2, 1),
    lambda x: ma.monarch_attn_fwd_varlen(x, x, x, x, x, 2, 2, 1),
    lambda x: ma.monarch_attn_fwd_prepad(x, x, x, x, 2, 2, 1),
    lambda x: ma.monarch_attn_fwd_objective(x, x, x, x, x, 2, 2, 1),
    lambda x: ma.monarch_attn_exact_fwd(x, x, x, x),
    lambda x: ma.monarch_attn_bwd(x, x, x, x, x, x, x, 2, 2, 1),
    lambda x: ma.monarch_attn_bwd_varlen(x, x, x, x, x, x, x, x, 2, 2, 1),
])
@pytest.mark.parametrize("x", [None, 3, torch.zeros(1, 1, 4, 8)])
def test_only_device_tensors(call, x):
    with pytest.raises(TypeError, match="q must be a device tensor"):
        call(x)


def test_refused_dtypes():
    with pytest.raises(TypeError):
        ma.dtype_code(torch.float64)
    assert ma.dtype_code(torch.bfloat16) == ma.MA_BF16


# ---- one argument at a time (on host tensors that say they are device tensors; the library is replaced) ----

class _Tensor(torch.Tensor):
    is_cuda = True


class _Library:
    def __getattr__(self, name):
        def reached(*args):
            raise AssertionError(f"{name} reached")

        return reached


SHAPE = (2, 3, 4, 8)
FORWARD, GRADIENT = ("q", "k", "v", "out"), ("q", "k", "v", "dout", "dq", "dk", "dv")
# entry point, its tensors of q's form, its other tensors, the call on all of them
ENTRIES = [
    (FORWARD, (), lambda q, k, v, out: ma.monarch_attn_fwd(q, k, v, out, 2, 2, 1)),
    (FORWARD, (), lambda q, k, v, out: ma.monarch_attn_fwd_noalloc(q, k, v, out, 2, 2, 1)),
    (FORWARD, ("lens",), lambda q, k, v, out, lens: ma.monarch_attn_fwd_varlen(q, k, v, out, lens, 2, 2, 1)),
    (FORWARD, ("lens",), lambda q, k, v, out, lens: ma.monarch_attn_fwd_prepad(q, k, v, out, 2, 2, 1, lens)),
    (FORWARD, ("obj",), lambda q, k, v, out, obj: ma.monarch_attn_fwd_objective(q, k, v, out, obj, 2, 2, 1)),
    (FORWARD, ("lse",), lambda q, k, v, out, lse: ma.monarch_attn_exact_fwd(q, k, v, out, lse)),
    (GRADIENT, (), lambda **t: ma.monarch_attn_bwd(*t.values(), 2, 2, 1)),
    (GRADIENT, ("lens",), lambda **t: ma.monarch_attn_bwd_varlen(*t.values(), 2, 2, 1)),
]
NAMES = ["fwd", "noalloc", "varlen", "prepad", "objective", "exact", "bwd", "bwd_varlen"]
EXTRA = {"lens": ((2,), torch.int32), "obj": ((2, 3, 1), torch.float32), "lse": ((2, 3, 4), torch.float32)}


def _tensor(shape, dtype, device="cpu"):
    return torch.zeros(shape, dtype=dtype, device=device).as_subclass(_Tensor)


def _arguments(names, extra):
    args = {name: _tensor(SHAPE, torch.bfloat16) for name in names}
    args.update({name: _tensor(*EXTRA[name]) for name in extra})
    return args


@pytest.fixture
def no_library(monkeypatch):
    from paper_2505_18698_amd import _binding

    monkeypatch.setattr(_binding, "LIB", _Library())
    monkeypatch.setattr(_binding._torch(), "current_device", lambda: None)
    monkeypatch.setattr(_binding._torch(), "current_stream", lambda index: 0)


@pytest.mark.parametrize("entry", ENTRIES, ids=NAMES)
def test_matching_tensors_reach_the_library(no_library, entry):
    names, extra, call = entry
    with pytest.raises(AssertionError, match="reached"):
        call(**_arguments(names, extra))


def _spoilt(shape, dtype):
    """A tensor of `shape` and `dtype` with one property wrong, and the exception for it."""
    other = torch.float16 if dtype == torch.bfloat16 else torch.int64
    strided = torch.zeros(*shape[:-1], 2 * shape[-1], dtype=dtype).as_subclass(_Tensor)[..., ::2]
    return {
        "none": (None, TypeError),
        "host": (torch.zeros(shape, dtype=dtype, device="meta"), TypeError),  # no device tensor, and not where q is
        "dtype": (_tensor(shape, other), ValueError),
        "short": (_tensor((*shape[:-1], shape[-1] - 1), dtype), ValueError),
        "rows": (_tensor((*shape[:-2], shape[-2] - 1, shape[-1]), dtype) if len(shape) > 1 else _tensor((1,), dtype), ValueError),
        "flat": (_tensor((*shape[:-2], shape[-2] * shape[-1]), dtype) if len(shape) > 1 else _tensor((), dtype), ValueError),
        "strided": (strided, ValueError),
        "device": (_tensor(shape, dtype, "meta"), ValueError),
    }


@pytest.mark.parametrize("fault", list(_spoilt(SHAPE, torch.bfloat16)))
@pytest.mark.parametrize("entry", ENTRIES, ids=NAMES)
def test_each_tensor_is_checked(no_library, entry, fault):
    """Every tensor but q, spoilt by itself, is refused by name before the library is called."""
    names, _, call = entry
    for name in names[1:]:
        args = _arguments(names, entry[1])
        args[name], error = _spoilt(SHAPE, torch.bfloat16)[fault]
        with pytest.raises(error, match=f"^{name} must "):
            call(**args)


@pytest.mark.parametrize("fault", ["none", "host", "flat", "strided"])
@pytest.mark.parametrize("entry", ENTRIES, ids=NAMES)
def test_q_is_checked(no_library, entry, fault):
    names, extra, call = entry
    args = _arguments(names, extra)
    args["q"], error = _spoilt(SHAPE, torch.bfloat16)[fault]
    with pytest.raises(error, match="^q must "):
        call(**args)


@pytest.mark.parametrize("fault", ["dtype", "short", "rows", "flat", "strided", "device"])
@pytest.mark.parametrize("entry", [e for e in ENTRIES if e[1]], ids=[n for n, e in zip(NAMES, ENTRIES) if e[1]])
def test_lengths_objective_and_logsumexp_are_checked(no_library, entry, fault):
    names, (extra,), call = entry
    args = _arguments(names, (extra,))
    args[extra] = _spoilt(*EXTRA[extra])[fault][0]
    with pytest.raises(ValueError, match=f"^{extra} must "):
        call(**args)
