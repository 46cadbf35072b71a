"""bf16 conv1d with the input read in place, position by position through LDS (pgk_conv_bf16.hip): each height of the tile, one to
three groups of positions, the weights of a block at once and in parts, the ends of rows, channels off the blocks, strides;
against the oracle.  Integers must come out exactly (sums exact in fp32, rounded once to bf16)."""
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


# B, Cin, L, Cout, Kw, stride, pad, dilation (two with few outputs and channels are the views', which are the faster way there)
CASES = [
    # up to 32 output channels: one, two and three groups of positions, one block of channels and several, whole and partly filled
    (20, 17, 2600, 18, 3, 1, 1, 1), (12, 64, 1025, 32, 1, 1, 0, 1), (10, 90, 1537, 31, 3, 2, 0, 2), (14, 33, 900, 24, 10, 1, 4, 1),
    # up to 64
    (30, 20, 3001, 64, 3, 1, 1, 1), (16, 96, 4097, 60, 5, 2, 2, 1), (24, 31, 2049, 64, 1, 2, 0, 1), (16, 100, 3000, 190, 10, 1, 9, 2),
    # more
    (40, 20, 2700, 202, 3, 1, 1, 1), (30, 66, 2100, 257, 5, 2, 2, 2), (40, 24, 2000, 128, 1, 1, 0, 1), (20, 40, 3001, 384, 7, 1, 3, 1),
    # rows shorter than a tile, padding wider than the row, halos and strides at their widest, rows of two elements
    (30, 16, 18, 40, 3, 1, 1, 1), (20, 24, 30, 33, 5, 1, 70, 9), (9, 40, 1500, 20, 2, 1, 0, 255), (9, 17, 1300, 40, 1, 3, 0, 1), (6, 48, 2, 32, 3, 1, 10, 1),
    # one workgroup
    (1, 16, 130, 16, 3, 1, 1, 1), (1, 37, 64, 20, 4, 1, 0, 1),
]


# Each instance of the kernel, (output channels of a tile, groups of 128 positions, weights of a block in parts), which test_kernels_reached_cpu.py
# asserts: one block of channels and several, whole and partly filled, ends of rows, strides, with the padding wider than the row
INSTANCES = [
    ((32, 1, False), (1, 18, 16, 18, 1, 1, 0, 2)), ((32, 1, False), (1, 33, 44, 35, 1, 1, 5, 1)), ((32, 1, False), (1, 79, 17, 71, 1, 1, 1, 2)), ((32, 1, False), (1, 29, 2, 17, 1, 1, 19, 3)),
    ((32, 2, False), (1, 20, 2, 16, 1, 2, 18, 3)), ((32, 2, False), (1, 48, 2, 35, 1, 2, 15, 3)), ((32, 2, False), (1, 96, 50, 35, 1, 2, 1, 3)),
    ((32, 2, True), (1, 17, 40, 20, 10, 1, 0, 1)), ((32, 2, True), (1, 47, 50, 36, 12, 1, 22, 2)), ((32, 2, True), (1, 84, 2, 26, 10, 1, 12, 1)),
    ((32, 3, False), (1, 18, 22, 23, 1, 3, 23, 3)), ((32, 3, False), (1, 45, 63, 33, 1, 3, 1, 2)), ((32, 3, False), (1, 70, 52, 36, 1, 3, 1, 1)),
    ((32, 3, True), (1, 38, 49, 40, 2, 3, 26, 2)), ((32, 3, True), (1, 28, 51, 19, 3, 3, 1, 1)), ((32, 3, True), (1, 30, 2, 35, 10, 2, 20, 1)), ((32, 3, True), (1, 82, 61, 35, 10, 2, 18, 1)),
    ((64, 1, False), (43, 48, 2091, 34, 1, 1, 1, 163)), ((64, 1, False), (15, 32, 3032, 103, 1, 1, 0, 1)), ((64, 1, False), (5, 102, 1572, 357, 1, 1, 59, 1)),
    ((64, 2, False), (43, 25, 2186, 34, 1, 2, 0, 9)), ((64, 2, False), (54, 34, 28, 476, 2, 1, 1, 3)), ((64, 2, False), (40, 81, 778, 133, 1, 2, 1, 3)),
    ((64, 2, True), (52, 16, 191, 438, 10, 1, 1, 3)), ((64, 2, True), (37, 48, 1421, 46, 10, 1, 33, 9)),
    ((64, 3, False), (1, 48, 59, 45, 3, 3, 1, 1)), ((64, 3, False), (1, 88, 1171, 37, 4, 2, 1, 40)), ((64, 3, False), (56, 29, 164, 130, 3, 2, 0, 64)),
    ((64, 3, True), (1, 32, 33, 46, 7, 2, 60, 20)), ((64, 3, True), (2, 20, 268, 30, 7, 1, 0, 41)), ((64, 3, True), (1, 77, 223, 43, 7, 1, 0, 34)),
    ((64, 3, True), (13, 64, 4673, 128, 7, 2, 0, 1)),
    ((128, 1, False), (37, 32, 1451, 118, 1, 1, 0, 1)), ((128, 1, False), (7, 35, 3855, 225, 1, 1, 7, 1)), ((128, 1, False), (51, 65, 1071, 100, 1, 1, 2, 1)),
    ((128, 2, False), (35, 21, 892, 368, 1, 2, 0, 37)), ((128, 2, False), (53, 30, 1636, 235, 1, 2, 5, 1)), ((128, 2, False), (39, 48, 3146, 92, 1, 2, 0, 1)),
    ((128, 2, True), (46, 17, 1732, 109, 4, 1, 4, 3)), ((128, 2, True), (38, 44, 1350, 98, 5, 1, 9, 9)),
    ((128, 3, False), (17, 32, 3772, 368, 1, 3, 1, 2)), ((128, 3, False), (35, 56, 2460, 237, 1, 3, 0, 3)), ((128, 3, False), (46, 85, 2155, 105, 2, 2, 0, 73)),
    ((128, 3, True), (25, 19, 1996, 327, 3, 3, 8, 1)), ((128, 3, True), (44, 48, 2601, 97, 3, 2, 63, 3)), ((128, 3, True), (59, 70, 1507, 70, 3, 1, 30, 127)),
    # 384 positions exactly, the last of three groups whole (also 28 channels above)
    ((64, 3, False), (1, 48, 59, 45, 3, 3, 1, 1)), ((128, 3, True), (34, 19, 3329, 499, 3, 3, 0, 1)),
]


def bf16(t):
    import torch
    return torch.from_numpy(t.view(np.int16)).cuda().view(torch.bfloat16)


def shifted(t, start):
    return bf16(np.concatenate([t.reshape(-1)[:start], t.reshape(-1)]))[start:].view(*t.shape)


@pytest.mark.parametrize("case", CASES)
def test_against_the_oracle(pgk, oracle, case):
    import torch
    B, Cin, L, Cout, Kw, stride, pad, dilation = case
    x = gen.small_ints(gen.tensor_seed(94, 1, L), B * Cin * L).reshape(B, Cin, L)
    w = gen.small_ints(gen.tensor_seed(94, 2, L), Cout * Cin * Kw).reshape(Cout, Cin, Kw)
    ref = oracle.conv1d(gen.f32_to_bf16_bits(x), gen.f32_to_bf16_bits(w), None, NONE, stride, pad, dilation)
    want = gen.bf16_bits_to_f32(gen.f32_to_bf16_bits(ref.astype(np.float32)))
    for start in (0, 1):
        got = pgk.conv1d(shifted(gen.f32_to_bf16_bits(x), start), bf16(gen.f32_to_bf16_bits(w)), None, NONE, stride, pad, dilation)
        torch.cuda.synchronize()
        assert np.array_equal(got.float().cpu().numpy(), want), (case, start)
    # a product of two bf16 values is exact in fp32 and K of them round at most K times by 2^-24 of sum |w x|; the
    # activation's slope is at most 1.13, it is good to a few units of 2^-24, and the output is rounded to 8 bits
    xs, ws = gen.uniform(gen.tensor_seed(94, 3, L), B * Cin * L, -1.0, 1.0), gen.normal(gen.tensor_seed(94, 4, L), Cout * Cin * Kw, (Cin * Kw) ** -0.5)
    xb, wb = gen.f32_to_bf16_bits(xs.reshape(B, Cin, L)), gen.f32_to_bf16_bits(ws.reshape(Cout, Cin, Kw))
    bias = gen.normal(gen.tensor_seed(94, 5, L), Cout, 0.5)
    scale = oracle.conv1d(xb & 0x7fff, wb & 0x7fff, np.abs(bias), NONE, stride, pad, dilation)
    for act in (RELU, GELU, SILU):
        got = pgk.conv1d(bf16(xb), bf16(wb), torch.from_numpy(bias).cuda(), act, stride, pad, dilation).float().cpu().numpy().astype(np.float64)
        ref = oracle.conv1d(xb, wb, bias, act, stride, pad, dilation)
        bound = (Cin * Kw + 12) * 2.0 ** -24 * 1.13 * scale + 2.0 ** -8 * np.abs(ref) + 1e-30
        assert np.all(np.abs(got - ref) <= bound), (case, act)


def test_neighbours_do_not_show(pgk, oracle):
    """Rows of NaN beside a row, and in the channels that pad the last block, leave its results alone."""
    import torch
    for B, Cin, L, Cout, Kw, stride, pad, dilation in [(21, 17, 1000, 40, 3, 1, 1, 1), (11, 50, 999, 200, 7, 2, 5, 2), (31, 20, 300, 20, 5, 1, 4, 2)]:
        x = gen.small_ints(gen.tensor_seed(94, 6, L), B * Cin * L).reshape(B, Cin, L)
        w = gen.f32_to_bf16_bits(gen.small_ints(gen.tensor_seed(94, 7, L), Cout * Cin * Kw).reshape(Cout, Cin, Kw))
        ref = oracle.conv1d(gen.f32_to_bf16_bits(x), w, None, NONE, stride, pad, dilation)
        x[1::2] = np.nan
        got = pgk.conv1d(bf16(gen.f32_to_bf16_bits(x)), bf16(w), None, NONE, stride, pad, dilation)
        want = gen.bf16_bits_to_f32(gen.f32_to_bf16_bits(ref.astype(np.float32)))
        assert np.array_equal(got[0::2].float().cpu().numpy(), want[0::2])
        assert torch.isnan(got[1::2]).all()


def test_without_a_workspace(pgk):
    """Sizes that never needed a workspace run without one as before."""
    import ctypes

    import torch
    B, Cin, L, Cout, Kw = 8, 20, 2000, 40, 3
    x, w = (torch.randint(-2, 3, s, device="cuda").bfloat16() for s in ((B, Cin, L), (Cout, Cin, Kw)))
    assert pgk.conv1d_workspace_bytes(B, Cin, L, Cout, Kw, 1, 1, 1, gen.BF16) >= Cout * Kw * 32 * 2
    y, z = pgk.conv1d(x, w, None, NONE, 1, 1, 1), torch.empty((B, Cout, L), dtype=torch.bfloat16, device="cuda")
    rc = pgk.load_library().pgk_conv1d(x.data_ptr(), w.data_ptr(), None, z.data_ptr(), B, Cin, L, Cout, Kw, 1, 1, 1, NONE, gen.BF16, None,
                                       ctypes.c_size_t(0), torch.cuda.current_stream().cuda_stream or None)
    torch.cuda.synchronize()
    assert rc == 0 and torch.equal(y, z)


def test_replays_of_a_graph(pgk):
    import torch
    x, w = torch.empty((12, 40, 2000), dtype=torch.bfloat16, device="cuda"), torch.empty((50, 40, 5), device="cuda").uniform_(-1, 1).bfloat16()
    s, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        x.uniform_(-1, 1)
        s.synchronize()
        with torch.cuda.graph(g, stream=s):
            y = pgk.conv1d(x, w, None, RELU, 2, 2, 1)
    for _ in range(3):
        x.uniform_(-1, 1)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, pgk.conv1d(x, w, None, RELU, 2, 2, 1))


def test_threads_with_different_needs_of_lds(pgk):
    """Calls that share a kernel and differ in the LDS they take (6 and 7 taps of 64 rows: 65 and 73 KB), from several threads."""
    import threading

    import torch
    x = torch.randint(-2, 3, (31, 17, 1862), device="cuda").bfloat16()
    weights = [torch.randint(-2, 3, (39, 17, Kw), device="cuda").bfloat16() for Kw in (6, 7)]
    want = [pgk.conv1d(x, w, None, NONE, 1, 0, 1) for w in weights]
    torch.cuda.synchronize()
    wrong = []

    def work(first):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for k in range(40):
                    which = (first + k) % 2
                    y = pgk.conv1d(x, weights[which], None, NONE, 1, 0, 1)
                    torch.cuda.current_stream().synchronize()
                    if not torch.equal(y, want[which]):
                        wrong.append((first, k))
        except Exception as e:
            wrong.append(e)
    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong, wrong[:3]


@pytest.mark.parametrize("instance,case", INSTANCES)
def test_instances(pgk, instance, case):
    """Integers exactly, from even and odd starts; uniform values within the bound of test_against_the_oracle."""
    import torch
    B, Cin, L, Cout, Kw, stride, pad, dilation = case
    g = torch.Generator(device="cuda").manual_seed(Cin * Kw)

    def in_64_bits(x, w, bias):
        xp = torch.nn.functional.pad(x.double(), (pad, pad))
        lout = (L + 2 * pad - dilation * (Kw - 1) - 1) // stride + 1
        y = bias.double().view(1, -1, 1).expand(B, -1, lout).clone()
        for b in range(B):
            for k in range(Kw):
                y[b] += w[:, :, k].double().contiguous() @ xp[b, :, k * dilation:k * dilation + (lout - 1) * stride + 1:stride].contiguous()
        return y
    x = torch.randint(-3, 4, (B, Cin, L), generator=g, device="cuda").bfloat16()
    w = torch.randint(-3, 4, (Cout, Cin, Kw), generator=g, device="cuda").bfloat16()
    bias = torch.randint(-7, 8, (Cout,), generator=g, device="cuda").float()
    want = in_64_bits(x, w, bias).float().bfloat16()
    for start in (0, 1):
        placed = torch.cat([x.new_full((start,), float("nan")), x.reshape(-1)])[start:].view(x.shape)
        assert torch.equal(pgk.conv1d(placed, w, bias, NONE, stride, pad, dilation), want), start
    x = torch.empty((B, Cin, L), device="cuda").uniform_(-1, 1, generator=g).bfloat16()
    w = torch.empty((Cout, Cin, Kw), device="cuda").normal_(0, (Cin * Kw) ** -0.5, generator=g).bfloat16()
    bias = torch.empty(Cout, device="cuda").normal_(0, 0.5, generator=g)
    got = pgk.conv1d(x, w, bias, SILU, stride, pad, dilation).double()
    ref = in_64_bits(x, w, bias)
    ref, scale = ref * torch.sigmoid(ref), in_64_bits(x.abs(), w.abs(), bias.abs())
    assert bool(((got - ref).abs() <= (Cin * Kw + 12) * 2.0 ** -24 * 1.13 * scale + 2.0 ** -8 * ref.abs() + 1e-30).all())
