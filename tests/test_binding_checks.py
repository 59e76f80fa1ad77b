"""The binding's argument checks (no GPU): what is not a device tensor is
refused with its name, on every entry point that takes tensors."""
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
