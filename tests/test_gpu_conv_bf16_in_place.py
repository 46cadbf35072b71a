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


# B, Cin, L, Cout, Kw, stride, pad, dilation
CASES = [
    # 32 output channels: one, two and three groups of positions, one block of channels and several, whole and partly filled
    (20, 17, 2600, 18, 3, 1, 1, 1), (12, 64, 1025, 32, 1, 1, 0, 1), (10, 90, 1537, 31, 3, 2, 0, 2), (14, 33, 900, 24, 10, 1, 4, 1),
    # 64
    (30, 20, 3001, 64, 3, 1, 1, 1), (16, 96, 4097, 60, 5, 2, 2, 1), (24, 31, 2049, 64, 1, 2, 0, 1), (16, 100, 3000, 190, 10, 1, 9, 2),
    # 128
    (40, 20, 2700, 202, 3, 1, 1, 1), (30, 66, 2100, 257, 5, 2, 2, 2), (40, 24, 2000, 128, 1, 1, 0, 1), (20, 40, 3001, 384, 7, 1, 3, 1),
    # rows shorter than a tile, padding wider than the row, halos and strides at their widest, rows of two elements
    (30, 16, 18, 40, 3, 1, 1, 1), (20, 24, 30, 33, 5, 1, 70, 9), (9, 40, 1500, 20, 2, 1, 0, 255), (9, 17, 1300, 40, 1, 3, 0, 1), (6, 48, 2, 32, 3, 1, 10, 1),
    # one workgroup
    (1, 16, 130, 16, 3, 1, 1, 1), (1, 37, 64, 20, 4, 1, 0, 1),
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
    x = torch.randint(-2, 3, (8, 384, 9000), device="cuda").bfloat16()
    weights = [torch.randint(-2, 3, (64, 384, Kw), device="cuda").bfloat16() for Kw in (6, 7)]
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
