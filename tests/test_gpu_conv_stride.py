"""Strided convolutions on the matrix-core path at the strides where the copies of the input are shared out
differently among workgroups (all phases in a thread, a few, one), with few and with many copies, against the oracle."""
import pytest

from paper_2511_06345_amd import inputs as gen
from util import TOL, c_to_numpy, rel_err, to_device

pytestmark = pytest.mark.gpu
F32, BF16 = gen.F32, gen.BF16

# B, Cin, L, Cout, Kw, stride, pad, dilation
CASES = [(1, 64, 301, 20, 3, 3, 1, 1),          # few workgroups: a phase each
         (2, 64, 4003, 33, 7, 5, 2, 1),         # groups that do not divide the phases
         (1, 64, 1500, 32, 20, 16, 9, 1), (1, 40, 3300, 17, 5, 32, 0, 7),
         (1, 64, 1500, 32, 32, 33, 16, 1), (1, 64, 2000, 16, 8, 64, 3, 9),
         (24, 64, 9000, 40, 32, 40, 0, 1),      # many workgroups: all phases in a thread
         (1, 64, 2100, 32, 4, 65, 1, 1), (2, 40, 8000, 32, 32, 160, 17, 1)]


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("case", CASES)
def test_strided(oracle, dtype, case):
    import torch
    from paper_2511_06345_amd import binding as pgk
    B, Cin, L, Cout, Kw, stride, pad, dil = case
    x = gen.uniform(gen.tensor_seed(94, 1, L), B * Cin * L, -1.0, 1.0).reshape(B, Cin, L)
    w = gen.normal(gen.tensor_seed(94, 2, L), Cout * Cin * Kw, (Cin * Kw) ** -0.5).reshape(Cout, Cin, Kw)
    bias = gen.normal(gen.tensor_seed(94, 3, L), Cout, 0.3)
    if dtype == BF16:
        x, w = gen.f32_to_bf16_bits(x), gen.f32_to_bf16_bits(w)
    assert pgk.conv1d_workspace_bytes(B, Cin, L, Cout, Kw, stride, pad, dil, dtype) > 0
    y = pgk.conv1d(to_device(x, dtype), to_device(w, dtype), torch.from_numpy(bias).cuda(), gen.ACT_RELU, stride, pad, dil)
    ref = oracle.conv1d(x, w, bias, gen.ACT_RELU, stride, pad, dil)
    assert y.shape == ref.shape
    assert rel_err(c_to_numpy(y, dtype), ref) <= TOL[dtype]
