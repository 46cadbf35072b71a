"""bf16 operands whose rows start on 2-byte boundaries only, copied through registers: odd K, odd N of
a plain B, both, and a convolution's taps at odd offsets, at the edges of tiles, with a partial last
K tile and none, one K tile to many, batches, and values behind the operands that must not be read
into a result."""
import numpy as np
import pytest
import torch

from paper_2511_06345_amd.inputs import ACT_NONE, ACT_SILU, BF16

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pgk():
    from paper_2511_06345_amd import binding
    binding.load_library()
    return binding


def _inside(values, offset=0):
    """The values as the middle of a buffer of NaN, `offset` elements from a 16-byte boundary on."""
    buf = torch.full((values.numel() + 64,), float("nan"), dtype=values.dtype, device="cuda")
    view = buf[32 + offset:32 + offset + values.numel()].view(values.shape)
    view.copy_(values)
    return view


def _copied(pgk, M, N, K, batch, bt):
    """Whether the call asks for padded copies of operands: for more than its partial products."""
    need = pgk.gemm_fused_workspace_bytes(M, N, K, batch, BF16, pgk.WS_B_TRANSPOSED if bt else 0)
    slices = pgk.gemm_plan(M, N, K, batch, BF16, bt)["slices"]
    return need != (0 if slices == 1 else -(-slices * batch * M * N * 4 // 256) * 256)


# integer values below 8 keep every sum exact in float32 (49 K < 2^24): the outputs are those of 64-bit
# sums rounded once to bf16, whatever the order
def _exact(pgk, M, N, K, batch, bt):
    g = torch.Generator(device="cuda").manual_seed(M * N + K)
    A = torch.randint(-7, 8, (batch, M, K), generator=g, device="cuda").to(torch.bfloat16)
    B = torch.randint(-7, 8, (batch, N, K) if bt else (batch, K, N), generator=g, device="cuda").to(torch.bfloat16)
    call = pgk.gemm_fused_bt if bt else pgk.gemm_fused
    C, rs = call(_inside(A), _inside(B), None, ACT_NONE, rowsum=True)
    ref = torch.stack([A[b].double() @ (B[b].double().t() if bt else B[b].double()) for b in range(batch)])
    assert torch.equal(C, ref.to(torch.bfloat16))
    # (row sums of integers: exact while below 2^24)
    if 49 * K * N < 2 ** 24 * 16:
        assert torch.allclose(rs.double(), ref.sum(-1), rtol=1e-6, atol=0.5)


@pytest.mark.parametrize("M,N,K,batch,bt", [
    (512, 2049, 64, 1, False),       # odd N, one whole K tile
    (300, 1501, 128, 2, False),      # odd N, whole K tiles, a batch whose entries start on odd elements
    (257, 4097, 190, 1, False),      # odd N, partial K tile
    (1024, 2304, 67, 1, False),      # odd K: A alone
    (1000, 2303, 129, 1, False),     # both; one K value in the last tile
    (2047, 1025, 703, 1, False),     # both, many tiles
    (130, 2100, 255, 3, True),       # transposed B, odd K
    (1000, 2303, 575, 1, True),
    (40, 40, 40001, 12, True),       # split along K
    (64, 4099, 200, 1, False),       # few rows
])
def test_odd_rows_exact(pgk, M, N, K, batch, bt):
    assert not _copied(pgk, M, N, K, batch, bt), "no copies of operands"
    _exact(pgk, M, N, K, batch, bt)


@pytest.mark.parametrize("M,N,K,batch,bt", [(1024, 2048, 1023, 1, True), (33, 33, 40001, 1, True), (64, 2051, 1000, 1, False)])
def test_odd_rows_copied_first_exact(pgk, M, N, K, batch, bt):
    assert _copied(pgk, M, N, K, batch, bt)
    _exact(pgk, M, N, K, batch, bt)


# every instance at one, two, three and many K tiles, whole and partial last ones
LARGE_A = [(600, 16400, 63), (600, 16400, 127), (3900, 4100, 129), (3900, 4100, 577), (2255, 6400, 487)]
LARGE_B = [(500, 50257, 64), (500, 50257, 62), (500, 50257, 128), (500, 50257, 190), (300, 20001, 640), (500, 50257, 646)]
SMALL = [(1000, 2303, 63), (1000, 2303, 65), (1000, 2303, 191), (1000, 2303, 575), (3000, 4999, 129)]
INSTANCES = ([(256, *s, 1, False) for s in LARGE_A + LARGE_B] + [(128, *s, 1, bt) for s in SMALL for bt in (False, True)] +
             [(128, 4096, 300, 255, 8, True), (128, 1000, 2303, 64, 1, False), (128, 200, 3001, 384, 4, False), (128, 90, 130, 36001, 6, True)])


@pytest.mark.parametrize("tile,M,N,K,batch,bt", INSTANCES)
def test_every_instance_exact(pgk, tile, M, N, K, batch, bt):
    assert pgk.gemm_plan(M, N, K, batch, BF16, bt)["tile"][:2] == (tile, tile) and not _copied(pgk, M, N, K, batch, bt)
    _exact(pgk, M, N, K, batch, bt)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("offset", [1, 2, 3])
@pytest.mark.parametrize("B,Cin,L,Cout,Kw,pad,dil", [(2, 64, 1001, 64, 3, 2, 2), (1, 64, 1002, 128, 1, 0, 1), (1, 128, 515, 256, 3, 1, 1)])
def test_convolution_of_an_input_on_any_element_exact(pgk, dtype, offset, B, Cin, L, Cout, Kw, pad, dil):
    g = torch.Generator(device="cuda").manual_seed(L)
    x = torch.randint(-7, 8, (B, Cin, L), generator=g, device="cuda").to(dtype)
    w = torch.randint(-7, 8, (Cout, Cin, Kw), generator=g, device="cuda").to(dtype)
    y = pgk.conv1d(_inside(x, offset), w, None, ACT_NONE, 1, pad, dil)
    xp = torch.nn.functional.pad(x.double(), (pad, pad))
    ref = torch.stack([sum(w[:, :, k].double() @ xp[b, :, k * dil:k * dil + y.shape[2]].contiguous() for k in range(Kw)) for b in range(B)])
    assert torch.equal(y, ref.to(dtype))


@pytest.mark.parametrize("B,Cin,L,Cout,Kw,pad,dil", [
    (2, 64, 1000, 64, 3, 1, 1), (1, 128, 4096, 256, 3, 1, 1), (2, 64, 777, 100, 5, 2, 1), (1, 64, 513, 48, 4, 0, 1),
    (3, 192, 300, 130, 3, 3, 3), (1, 64, 129, 64, 7, 3, 1), (1, 64, 2001, 512, 1, 0, 1), (2, 64, 640, 64, 3, 101, 1),
    # large grids (most of these read their input in place, through LDS: sizes that reach each tile through registers are in
    # test_gpu_register_trips.py, asserted by test_kernels_reached_cpu.py)
    (8, 128, 4097, 512, 3, 1, 1), (9, 64, 4001, 500, 5, 2, 1), (97, 64, 101, 512, 3, 1, 1), (49, 128, 130, 1000, 3, 0, 1),
    (12, 64, 4097, 128, 3, 1, 1), (13, 128, 3900, 100, 7, 3, 1),
])
def test_convolution_taps_at_odd_offsets_exact(pgk, B, Cin, L, Cout, Kw, pad, dil):
    g = torch.Generator(device="cuda").manual_seed(L + Cout)
    x = torch.randint(-7, 8, (B, Cin, L), generator=g, device="cuda").to(torch.bfloat16)
    w = torch.randint(-7, 8, (Cout, Cin, Kw), generator=g, device="cuda").to(torch.bfloat16)
    bias = torch.randint(-7, 8, (Cout,), generator=g, device="cuda").float()
    y = pgk.conv1d(_inside(x), _inside(w), bias, ACT_NONE, 1, pad, dil)
    Lout = y.shape[2]
    xp = torch.nn.functional.pad(x.double(), (pad, pad))
    ref = bias.double().view(1, -1, 1).expand(B, -1, Lout).clone()
    for b in range(B):
        for k in range(Kw):
            ref[b] += w[:, :, k].double() @ xp[b, :, k * dil:k * dil + Lout].contiguous()
    assert torch.equal(y, ref.to(torch.bfloat16))


def test_activation_against_64_bits(pgk):
    rng = np.random.default_rng(7)
    M, N, K = 129, 1021, 515
    A = torch.from_numpy(rng.uniform(-1, 1, (1, M, K)).astype(np.float32)).to(torch.bfloat16)
    B = torch.from_numpy((rng.standard_normal((1, K, N)) / K ** 0.5).astype(np.float32)).to(torch.bfloat16)
    bias = torch.from_numpy(rng.standard_normal(N).astype(np.float32))
    C, _ = pgk.gemm_fused(A.cuda(), B.cuda(), bias.cuda(), ACT_SILU, rowsum=False)
    x = A.double() @ B.double() + bias.double()
    ref = x * torch.sigmoid(x)
    err = (C.cpu().double() - ref).abs() / torch.maximum(ref.abs(), ref.pow(2).mean().sqrt())
    # half a unit of the stored bf16 (2^-9) and the float32 sums
    assert err.max() < 2.0 ** -8


@pytest.mark.parametrize("M,N,K", [(256, 44864, 3079), (384, 30533, 361)])
def test_row_sums_are_no_less_exact_than_of_padded_operands(pgk, M, N, K):
    assert not _copied(pgk, M, N, K, 1, True)
    g = torch.Generator(device="cuda").manual_seed(K)
    A = torch.empty((1, M, K), device="cuda").uniform_(-1, 1, generator=g).to(torch.bfloat16)
    B = torch.empty((1, N, K), device="cuda").normal_(0, K ** -0.5, generator=g).to(torch.bfloat16)
    ref = (A[0].double() @ B[0].double().t()).sum(-1)
    pad = torch.nn.functional.pad
    odd, even = (pgk.gemm_fused_bt(x, y, None, ACT_NONE, rowsum=True)[1][0].double() for x, y in ((A, B), (pad(A, (0, 1)), pad(B, (0, 1)))))
    # (the errors of a few hundred rows: their norms agree to a tenth where both are sums of the same kind)
    assert float((odd - ref).norm()) <= 1.2 * float((even - ref).norm())


@pytest.mark.parametrize("M,N,K,batch,bt", [
    (1024, 2048, 1023, 1, True), (832, 1440, 379, 32, True), (2048, 2047, 320, 1, False), (700, 513, 511, 2, False), (4096, 4095, 512, 1, False),
    (4096, 4096, 511, 1, False),
    (32, 3072, 4429, 1, False), (9, 1000, 8191, 1, True),        # few rows
])
def test_without_room_for_copies_operands_are_read_in_place(pgk, M, N, K, batch, bt):
    assert _copied(pgk, M, N, K, batch, bt)
    g = torch.Generator(device="cuda").manual_seed(K)
    A = torch.randint(-7, 8, (batch, M, K), generator=g, device="cuda").to(torch.bfloat16)
    B = torch.randint(-7, 8, (batch, N, K) if bt else (batch, K, N), generator=g, device="cuda").to(torch.bfloat16)
    ws = torch.empty(16, dtype=torch.uint8, device="cuda")
    C, _ = (pgk.gemm_fused_bt if bt else pgk.gemm_fused)(_inside(A), _inside(B), None, ACT_NONE, rowsum=False, workspace=ws)
    ref = torch.stack([A[b].double() @ (B[b].double().t() if bt else B[b].double()) for b in range(batch)])
    assert torch.equal(C, ref.to(torch.bfloat16))


def test_split_call_with_room_for_its_partial_products_only(pgk):
    M, N, K, splits = 512, 500, 8191, 4
    q = pgk.gemm_splitk_workspace_bytes
    products = splits * M * N * 4
    assert q(M, N, K, 1, BF16, splits, 0) > products
    g = torch.Generator(device="cuda").manual_seed(3)
    A = torch.randint(-7, 8, (1, M, K), generator=g, device="cuda").to(torch.bfloat16)
    B = torch.randint(-7, 8, (1, K, N), generator=g, device="cuda").to(torch.bfloat16)
    ws = torch.full((products + 256,), 255, dtype=torch.uint8, device="cuda")
    C, _ = pgk.gemm_splitk(_inside(A), _inside(B), None, ACT_NONE, splits=splits, rowsum=False, workspace=ws[:products])
    assert torch.equal(C[0], (A[0].double() @ B[0].double()).to(torch.bfloat16))
    assert bool((ws[products:] == 255).all())
    with pytest.raises(pgk.PgkError):
        pgk.gemm_splitk(A, B, None, ACT_NONE, splits=splits, rowsum=False, workspace=ws[:products - 256])


def test_without_room_and_without_a_kernel_the_call_is_refused(pgk):
    A, B = torch.ones((1, 500, 1001), dtype=torch.bfloat16, device="cuda"), torch.ones((1, 30, 1001), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(pgk.PgkError):
        pgk.gemm_fused_bt(A, B, None, ACT_NONE, rowsum=False, workspace=torch.empty(16, dtype=torch.uint8, device="cuda"))


def test_convolution_without_room_for_copies_reads_its_input_in_place(pgk):
    # (through LDS at this size; through registers: test_convolution_without_room_for_copies_goes_through_registers)
    B, Cin, L, Cout, Kw, pad = 7, 384, 1656, 265, 10, 3
    need = pgk.conv1d_workspace_bytes(B, Cin, L, Cout, Kw, 1, pad, 1, BF16)
    assert need > 2 * 2 * B * Cin * L                       # two copies of the input
    g = torch.Generator(device="cuda").manual_seed(4)
    x = torch.randint(-3, 4, (B, Cin, L), generator=g, device="cuda").to(torch.bfloat16)
    w = torch.randint(-3, 4, (Cout, Cin, Kw), generator=g, device="cuda").to(torch.bfloat16)
    ws = torch.full((need,), 255, dtype=torch.uint8, device="cuda")
    y = pgk.conv1d(_inside(x), _inside(w), None, ACT_NONE, 1, pad, 1, workspace=ws[:need // 2])
    assert torch.equal(y, pgk.conv1d(x, w, None, ACT_NONE, 1, pad, 1))
    xp = torch.nn.functional.pad(x.double(), (pad, pad))
    ref = torch.stack([sum(w[:, :, k].double() @ xp[b, :, k:k + y.shape[2]].contiguous() for k in range(Kw)) for b in range(B)])
    assert torch.equal(y, ref.to(torch.bfloat16)) and bool((ws[need // 2:] == 255).all())
    with pytest.raises(pgk.PgkError):
        pgk.conv1d(x, w, None, ACT_NONE, 1, pad, 1, workspace=ws[:256])
