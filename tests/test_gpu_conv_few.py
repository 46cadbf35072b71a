"""Convolutions with few input channels (one kernel for the whole layer: input and weights in LDS, fp32
matrix instruction, stores straight from the accumulators) against the oracle, at the edges of its
tiles of 128 positions, blocks of channels, pairs of k and row alignments."""
import numpy as np
import pytest

from paper_2511_06345_amd import inputs as gen
from util import TOL, c_to_numpy, rel_err, to_device

gpu = pytest.mark.gpu
F32, BF16 = gen.F32, gen.BF16

# B, Cin, L, Cout, Kw, stride, pad, dilation
CASES = [(128, 1, 256, 16, 3, 1, 1, 1),          # two whole tiles, rows aligned
         (192, 1, 255, 33, 10, 1, 0, 1),         # an odd row length: windows moved, both ends cut
         (96, 3, 385, 70, 7, 1, 3, 1),           # three tiles and one position, K odd (21)
         (128, 2, 300, 5, 1, 1, 0, 1),           # one tap, fewer channels than waves
         (64, 1, 2600, 130, 10, 5, 2, 1),        # strided, two blocks of channels
         (40, 15, 1700, 140, 3, 1, 2, 2),        # 45 products per sum, the kernel's longest
         (128, 4, 768, 128, 6, 2, 5, 3),         # 24 products
         (24, 2, 1300, 32, 3, 1, 4096, 4096),    # a dilation that takes more than 64 KiB of LDS
         (74, 1, 1027, 512, 10, 1, 1, 1),        # every sixteenth channel (fp32, odd rows)
         (74, 1, 1027, 300, 16, 1, 1, 1)]        # ... with blocks only partly filled
SIXTEENTH = CASES[-2:]


def lout_of(case):
    B, Cin, L, Cout, Kw, stride, pad, dil = case
    return (L + 2 * pad - dil * (Kw - 1) - 1) // stride + 1


@pytest.mark.parametrize("case", CASES)
def test_cases_are_within_the_rule(case):
    """What the kernel asks for, restated: a case outside of it would run on the bounds-checked kernel."""
    B, Cin, L, Cout, Kw, stride, pad, dil = case
    K, Lout = Cin * Kw, lout_of(case)
    pairs = -(-Lout // 128) * -(-Cout // 128) * B
    assert Lout >= 64 and K <= 48 and (K <= 24 or Cout >= 128)
    assert pairs >= (1024 if K > 24 else 384 if K > 8 else 256)
    assert Cin * stride <= min(32, Cout // 2 + 4)
    K2 = (K + 1) // 2 * 2
    lds = Cin * ((128 + 14) * stride + (Kw - 1) * dil + 1) + K2 * 132 + 128 + K2
    assert lds <= 20 * 1024 and (lds * 4 > 65536) == (dil == 4096)
    sixteenth = Lout % 16 != 0 and Cout >= 256 and K2 <= 16 and Lout // 128 * -(-Cout // 512) * B >= 512
    assert sixteenth == (case in SIXTEENTH)


@pytest.fixture(scope="module")
def pgk():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2511_06345_amd import binding
    binding.load_library()
    return binding


@gpu
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


@gpu
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


@gpu
@pytest.mark.parametrize("case", [(11, 1, 30001, 256, 3, 1, 0, 1), (11, 1, 30002, 256, 10, 1, 4, 1), (7, 2, 118003, 512, 7, 5, 3, 1)])
def test_outputs_beyond_the_last_level_cache_are_exact(pgk, case):
    """fp32, every sixteenth channel and more than 300 MB of output: non-temporal stores.  Small integers: every sum exact."""
    import torch
    B, Cin, L, Cout, Kw, stride, pad, dil = case
    Lout = lout_of(case)
    assert B * Cout * Lout * 4 > 300e6 and Lout % 16 != 0 and Lout // 128 * -(-Cout // 512) * B >= 512
    g = torch.Generator(device="cuda").manual_seed(L)
    x = torch.randint(-7, 8, (B, Cin, L), generator=g, device="cuda").float()
    w = torch.randint(-7, 8, (Cout, Cin, Kw), generator=g, device="cuda").float()
    bias = torch.randint(-7, 8, (Cout,), generator=g, device="cuda").float()
    n = B * Cout * Lout
    flat = torch.full((n + 64,), 7.5, device="cuda")
    y = flat[17:17 + n].view(B, Cout, Lout)
    pgk.conv1d(x, w, bias, gen.ACT_NONE, stride, pad, dil, out=y)
    assert bool((flat[:17] == 7.5).all()) and bool((flat[17 + n:] == 7.5).all()), "wrote outside y"
    xp = torch.nn.functional.pad(x.double(), (pad, pad))
    span = (Lout - 1) * stride + 1
    for b in range(B):
        ref = bias.double().view(-1, 1) + sum(w[:, :, k].double() @ xp[b, :, k * dil:k * dil + span:stride].contiguous() for k in range(Kw))
        assert torch.equal(y[b].double(), ref), b
