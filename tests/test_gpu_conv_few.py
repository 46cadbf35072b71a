"""Convolutions with few input channels (one kernel for the whole layer: input and weights in LDS, fp32
matrix instruction, stores straight from the accumulators) against the oracle, at the edges of its
tiles of 128 positions, blocks of channels, pairs of k and row alignments."""
import numpy as np
import pytest

from paper_2511_06345_amd import inputs as gen
from util import TOL, c_to_numpy, rel_err, to_device

pytestmark = pytest.mark.gpu
F32, BF16 = gen.F32, gen.BF16

# B, Cin, L, Cout, Kw, stride, pad, dilation: at least 256 pairs of a tile and 128 channels each (1024
# for sums of more than 24 products)
CASES = [(128, 1, 256, 16, 3, 1, 1, 1),          # two whole tiles, rows aligned
         (128, 1, 255, 33, 10, 1, 0, 1),         # an odd row length: windows moved, both ends cut
         (90, 3, 385, 70, 7, 1, 3, 1),           # three tiles and one position, K odd (21)
         (128, 2, 300, 5, 1, 1, 0, 1),           # one tap, fewer channels than waves
         (64, 1, 2600, 130, 10, 5, 2, 1),        # strided, two blocks of channels
         (40, 15, 1700, 140, 3, 1, 2, 2),        # 45 products per sum, the kernel's longest
         (43, 4, 768, 128, 6, 2, 5, 3),          # 24 products
         (70, 1, 1027, 512, 10, 1, 1, 1),        # every sixteenth channel (fp32, odd rows)
         (70, 1, 1027, 300, 16, 1, 1, 1)]        # ... with blocks only partly filled


@pytest.fixture(scope="module")
def pgk():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2511_06345_amd import binding
    binding.load_library()
    return binding


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("case", CASES)
def test_few_channels_match_the_oracle_and_stay_in_bounds(pgk, oracle, dtype, case):
    import torch
    B, Cin, L, Cout, Kw, stride, pad, dil = case
    x = gen.uniform(gen.tensor_seed(97, 1, L), B * Cin * L, -1.0, 1.0).reshape(B, Cin, L)
    w = gen.normal(gen.tensor_seed(97, 2, L), Cout * Cin * Kw, (Cin * Kw) ** -0.5).reshape(Cout, Cin, Kw)
    bias = gen.normal(gen.tensor_seed(97, 3, L), Cout, 0.3)
    if dtype == BF16:
        x, w = gen.f32_to_bf16_bits(x), gen.f32_to_bf16_bits(w)
    assert pgk.conv1d_workspace_bytes(B, Cin, L, Cout, Kw, stride, pad, dil, dtype) == 0
    dx, dw, db = to_device(x, dtype), to_device(w, dtype), torch.from_numpy(bias).cuda()
    Lout = pgk.conv1d_out_len(L, Kw, stride, pad, dil)
    for act in (gen.ACT_NONE, gen.ACT_RELU, gen.ACT_GELU_TANH, gen.ACT_SILU):
        ref = oracle.conv1d(x, w, bias, act, stride, pad, dil)
        for start in (0, 1, 3):                  # y on any element
            n = B * Cout * Lout
            flat = torch.full((n + 64,), 7.0, dtype=dx.dtype, device="cuda")
            y = flat[16 + start:16 + start + n].view(B, Cout, Lout)
            pgk.conv1d(dx, dw, db, act, stride, pad, dil, out=y)
            torch.cuda.synchronize()
            assert rel_err(c_to_numpy(y, dtype), ref) <= TOL[dtype], (case, act, start)
            assert bool((flat[:16 + start] == 7.0).all()) and bool((flat[16 + start + n:] == 7.0).all()), "wrote outside y"


def test_few_channels_integers_are_exact_and_special_values_stay_in_place(pgk, oracle):
    """Small integers: every sum exact.  An infinity or NaN reaches the outputs whose window holds it
    and no other (the k that fills up a pair has a zero weight and must not meet it)."""
    import torch
    B, Cin, L, Cout, Kw = 64, 3, 700, 40, 7
    x = gen.small_ints(5, B * Cin * L).reshape(B, Cin, L)
    w = gen.small_ints(6, Cout * Cin * Kw).reshape(Cout, Cin, Kw)
    y = pgk.conv1d(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), None, gen.ACT_NONE, 1, 3, 1)
    assert np.array_equal(y.cpu().numpy().astype(np.float64), oracle.conv1d(x, w, None, gen.ACT_NONE, 1, 3, 1))
    x[3, 0, 0] = np.inf
    x[7, 2, 699] = np.nan
    y = pgk.conv1d(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), None, gen.ACT_NONE, 1, 3, 1).cpu().numpy()
    bad = ~np.isfinite(y)
    want = np.zeros((B, 700), dtype=bool)
    want[3, :4] = want[7, 696:] = True
    assert np.array_equal(bad.any(axis=1), want)
