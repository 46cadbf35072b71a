"""fp32 conv1d with the input and the weights read in place (pgk_gemm_f32_terms.h): each height of the tile, the ends of rows,
channels and positions off the tiles, sums off the K steps, strides; against the oracle.

Bound: a sum of K products is added in ceil(K / 32) + 2 roundings of 2^-24 of a partial sum, and each product is
within 2^-24 of itself, so |error| <= (K / 32 + 4) 2^-24 sum |w x| + the bias's and the activation's (as in test_gpu_f32_terms)."""
import numpy as np
import pytest

from paper_2511_06345_amd import inputs as gen

pytestmark = pytest.mark.gpu
NONE, RELU, GELU, SILU = gen.ACT_NONE, gen.ACT_RELU, gen.ACT_GELU_TANH, gen.ACT_SILU


@pytest.fixture(scope="module")
def pgk():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2511_06345_amd import binding
    binding.load_library()
    return binding


# B, Cin, L, Cout, Kw, stride, pad, dilation
CASES = [
    # tiles of 128 or 64 output channels, whole tiles and rows and one more or less of each; one, two and many K steps
    (30, 32, 2050, 128, 3, 1, 0, 1), (30, 33, 2049, 129, 3, 1, 1, 1), (9, 20, 3000, 383, 5, 1, 2, 1), (24, 7, 1400, 300, 4, 1, 0, 1),
    (28, 17, 2200, 102, 1, 1, 1, 2), (51, 38, 2302, 69, 1, 2, 5, 2), (39, 66, 1379, 67, 1, 1, 0, 1), (22, 34, 4624, 67, 3, 2, 5, 2),
    (50, 120, 902, 68, 2, 1, 5, 1),
    # of 64 or 32
    (20, 57, 1801, 64, 5, 1, 2, 1), (20, 31, 1700, 63, 1, 1, 0, 1), (12, 100, 1537, 192, 3, 2, 1, 1), (16, 40, 3001, 50, 3, 1, 2, 2),
    # of 32 (the last one is the views', the faster way there)
    (20, 53, 2500, 19, 3, 1, 1, 1), (24, 18, 1300, 32, 10, 1, 0, 1), (14, 37, 3300, 26, 5, 1, 2, 1), (10, 90, 1900, 30, 3, 2, 0, 2),
    # rows of less than a tile, padding wider than the row, wide halos, strides beyond the tap count, one channel (with five taps on the
    # bounds-checked kernel: too few products)
    (40, 16, 20, 24, 3, 1, 1, 1), (30, 24, 30, 40, 5, 1, 70, 9), (8, 24, 900, 40, 3, 7, 2, 40), (6, 5, 4001, 48, 9, 3, 4, 2), (3, 1, 700, 16, 5, 1, 2, 1),
    (3, 1, 700, 16, 13, 1, 2, 1), (9, 1, 900, 40, 20, 1, 5, 1), (11, 130, 1201, 128, 2, 1, 1, 1),
]


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("start", [0, 1])
def test_against_the_oracle(pgk, oracle, case, start):
    import torch
    B, Cin, L, Cout, Kw, stride, pad, dilation = case
    x = gen.uniform(gen.tensor_seed(95, 1, L), B * Cin * L, -1.0, 1.0).reshape(B, Cin, L)
    w = gen.normal(gen.tensor_seed(95, 2, L), Cout * Cin * Kw, 0.3).reshape(Cout, Cin, Kw)
    bias = gen.normal(gen.tensor_seed(95, 3, L), Cout, 0.5)

    def on_device(t):
        return torch.from_numpy(np.concatenate([t.reshape(-1)[:start], t.reshape(-1)])).cuda()[start:].view(*t.shape)
    for act, b in ((NONE, None), (GELU, bias)):
        got = pgk.conv1d(on_device(x), on_device(w), torch.from_numpy(b).cuda() if b is not None else None, act, stride, pad, dilation)
        torch.cuda.synchronize()
        ref = oracle.conv1d(x, w, b, act, stride, pad, dilation)
        scale = oracle.conv1d(np.abs(x), np.abs(w), np.abs(b) if b is not None else None, NONE, stride, pad, dilation)
        # (GELU's slope is at most 1.13, and it is evaluated to a few units of 2^-24 of its argument)
        bound = (Cin * Kw / 32 + 4 + (8 if act else 0)) * 2.0 ** -24 * 1.13 * scale + 1e-30
        assert np.all(np.abs(got.cpu().numpy().astype(np.float64) - ref) <= bound), (case, act)


def test_integers_are_exact_and_ends_are_zero(pgk, oracle):
    """Sums of integers come out exactly; what lies beside a row, in the neighbouring rows, does not show (NaN there)."""
    import torch
    for B, Cin, L, Cout, Kw, stride, pad, dilation in [(30, 33, 1000, 70, 3, 1, 1, 1), (30, 33, 999, 30, 7, 2, 5, 2), (20, 50, 300, 129, 5, 1, 4, 2)]:
        x = gen.small_ints(gen.tensor_seed(95, 4, L), B * Cin * L).reshape(B, Cin, L)
        w = gen.small_ints(gen.tensor_seed(95, 5, L), Cout * Cin * Kw).reshape(Cout, Cin, Kw)
        ref = oracle.conv1d(x, w, None, NONE, stride, pad, dilation)
        got = pgk.conv1d(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), None, NONE, stride, pad, dilation)
        assert np.array_equal(got.cpu().numpy().astype(np.float64), ref)
        # a batch entry of NaN between the others
        y = x.copy()
        y[1::2] = np.nan
        got2 = pgk.conv1d(torch.from_numpy(y).cuda(), torch.from_numpy(w).cuda(), None, NONE, stride, pad, dilation)
        assert np.array_equal(got2[0::2].cpu().numpy().astype(np.float64), ref[0::2])
        assert torch.isnan(got2[1::2]).all()
        # infinities where fp32 has them: the tile is computed again with the fp32 instruction
        z = x.copy()
        z[0, 3, 51] = np.inf              # (an odd place: the strided case reads no others)
        got3 = pgk.conv1d(torch.from_numpy(z).cuda(), torch.from_numpy(np.abs(w) + 1).cuda(), None, NONE, stride, pad, dilation).cpu().numpy()
        ref3 = oracle.conv1d(z, np.abs(w) + 1, None, NONE, stride, pad, dilation)
        assert np.array_equal(np.isinf(got3), np.isinf(ref3)) and np.isinf(got3).any()
        fine = np.isfinite(ref3)
        assert np.array_equal(got3[fine].astype(np.float64), ref3[fine])


def test_replays_of_a_graph(pgk):
    """One launch and no copies: captured before anything has run, replayed on changing inputs."""
    import torch
    x = torch.empty((12, 40, 2000), device="cuda")
    w = torch.empty((50, 40, 5), device="cuda").uniform_(-1, 1)
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        x.uniform_(-1, 1)
        s.synchronize()
        with torch.cuda.graph(g, stream=s):
            y = pgk.conv1d(x, w, None, RELU, 1, 2, 1)
    for i in range(3):
        x.uniform_(-1, 1)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, pgk.conv1d(x, w, None, RELU, 1, 2, 1))


@pytest.mark.parametrize("Cin,Kw", [(1, 1), (2, 1), (1, 3), (5, 1), (3, 3), (11, 1)])
def test_short_sums_round_like_multiply_adds(pgk, Cin, Kw):
    """Sums of fewer than 12 products, heavy-tailed: each product's error is at most a rounding of it and of the sums that follow
    (a single product: correctly rounded)."""
    import torch
    for B, L, Cout in ((1, 300, 40), (2, 3001, 70)):
        g = torch.Generator(device="cuda").manual_seed(Cin * 10 + Kw)
        x, w = (torch.exp(4 * torch.randn(s, device="cuda", generator=g)) * torch.randn(s, device="cuda", generator=g).sign() for s in ((B, Cin, L), (Cout, Cin, Kw)))
        y = pgk.conv1d(x, w, None, NONE)
        taps = x.double().unfold(2, Kw, 1).permute(0, 1, 3, 2).reshape(B, Cin * Kw, -1)
        ref, scale = torch.matmul(w.double().reshape(Cout, -1), taps), torch.matmul(w.double().abs().reshape(Cout, -1), taps.abs())
        if Cin * Kw == 1:
            assert torch.equal(y, ref.float())
        assert bool(((y.double() - ref).abs() <= Cin * Kw * 2.0 ** -24 * scale).all())


def test_ordinary_calls_allocate_what_they_write_to(pgk):
    """No room for copies of the input that the way taken does not make (137 MB of them here; the weights regrouped for bf16 0.2 MB)."""
    import torch
    for dtype, (B, Cin, L, Cout, Kw, stride) in ((torch.float32, (4, 152, 53120, 19, 7, 1)), (torch.bfloat16, (8, 384, 11631, 61, 5, 2))):
        x, w = torch.zeros((B, Cin, L), dtype=dtype, device="cuda"), torch.zeros((Cout, Cin, Kw), dtype=dtype, device="cuda")
        code = gen.F32 if dtype == torch.float32 else gen.BF16
        assert pgk.conv1d_workspace_bytes(B, Cin, L, Cout, Kw, stride, 0, 1, code) > x.numel() * x.element_size() // 2
        lout = (L - Kw) // stride + 1
        for out in (None, torch.empty((B, Cout, lout), dtype=dtype, device="cuda")):
            torch.cuda.synchronize()
            torch.cuda.reset_peak_memory_stats()
            before = torch.cuda.memory_allocated()
            y = pgk.conv1d(x, w, None, RELU, stride, 0, 1, out=out)
            assert torch.cuda.max_memory_allocated() - before <= (y.numel() * y.element_size() if out is None else 0) + (1 << 20)
            del y
