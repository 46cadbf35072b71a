"""Products of few rows in one launch (all of K in a workgroup): both layouts of B, both types, the row counts
around a block of sixteen, columns around the workgroups' and the lanes' shares, K around a step and its
pieces, batches, operands on any element, and values around the operands that must not enter a result."""
import pytest
import torch

from paper_2511_06345_amd.inputs import ACT_GELU_TANH, ACT_NONE, ACT_RELU, ACT_SILU, BF16, F32

pytestmark = pytest.mark.gpu
TYPES = {F32: torch.float32, BF16: torch.bfloat16}


@pytest.fixture(scope="module")
def pgk():
    from paper_2511_06345_amd import binding
    binding.load_library()
    return binding


def _inside(values, offset):
    """The values in the middle of a buffer of NaN, `offset` elements from a 16-byte boundary on."""
    buf = torch.full((values.numel() + 64,), float("nan"), dtype=values.dtype, device="cuda")
    view = buf[32 + offset:32 + offset + values.numel()].view(values.shape)
    view.copy_(values)
    return view


def _one_pass(pgk, M, N, K, batch, dtype, bt):
    """No workspace but the row sums', whatever the alignment: the kernel for few rows."""
    flags = pgk.WS_UNALIGNED | (pgk.WS_B_TRANSPOSED if bt else 0)
    return pgk.gemm_fused_workspace_bytes(M, N, K, batch, dtype, flags) == 0 and \
        pgk.gemm_plan(M, N, K, batch, dtype, bt)["slices"] == 1


BT = [(1, 256, 64), (8, 4097, 128), (15, 301, 129), (16, 1000, 1023), (7, 4111, 2056), (3, 272, 65), (2, 5000, 136), (16, 4096, 100), (5, 4098, 8200), (5, 4098, 4096),
      (8, 1500, 128), (2, 1501, 264), (5, 4098, 8201), (16, 1000, 300)]
PLAIN = {BF16: [(1, 256, 64), (16, 4100, 33 * 32), (5, 4224, 1000), (9, 16385, 72), (15, 16501, 100), (3, 300, 1024),
                (31, 257, 65), (6, 2051, 8201), (20, 2101, 9000), (17, 2049, 96), (32, 16387, 71), (24, 4103, 259), (6, 6151, 8201), (20, 6101, 9000)],
         F32: [(1, 256, 64), (16, 257, 100), (8, 4097, 1040), (3, 4160, 2052), (9, 301, 1023), (15, 4099, 67), (2, 258, 515), (3, 8260, 8200), (3, 10240, 8192), (7, 10256, 2052)]}
CASES = [(d, *s, True) for d in (F32, BF16) for s in BT] + [(d, *s, False) for d in (F32, BF16) for s in PLAIN[d]]
# of these, left to the tiles: whatever the batch, and with three entries
OUTSIDE = {(F32, 5, 4098, 8200, True), (F32, 5, 4098, 8201, True), (BF16, 5, 4098, 8200, True), (F32, 3, 8260, 8200, False), (F32, 3, 4160, 2052, False), (BF16, 6, 2051, 8201, False), (BF16, 20, 2101, 9000, False),
           (BF16, 8, 4097, 128, True), (BF16, 2, 5000, 136, True), (BF16, 16, 4096, 100, True), (BF16, 8, 1500, 128, True)}
OUTSIDE_BATCHED = {(F32, 8, 4097, 128, True), (F32, 2, 5000, 136, True), (F32, 16, 4096, 100, True)}


@pytest.mark.parametrize("dtype,M,N,K,bt", CASES)
@pytest.mark.parametrize("batch,offset", [(1, 0), (3, 1)])
def test_integers_exact(pgk, dtype, M, N, K, bt, batch, offset):
    # |sum| <= 49 K < 2^24: exact in any order
    outside = OUTSIDE | OUTSIDE_BATCHED if batch > 1 else OUTSIDE
    assert _one_pass(pgk, M, N, K, batch, dtype, bt) == ((dtype, M, N, K, bt) not in outside)
    g = torch.Generator(device="cuda").manual_seed(M + N * K)
    A = torch.randint(-7, 8, (batch, M, K), generator=g, device="cuda").to(TYPES[dtype])
    B = torch.randint(-7, 8, (batch, N, K) if bt else (batch, K, N), generator=g, device="cuda").to(TYPES[dtype])
    bias = torch.randint(-7, 8, (N,), generator=g, device="cuda").float()
    call = pgk.gemm_fused_bt if bt else pgk.gemm_fused
    C, rs = call(_inside(A, offset), _inside(B, offset), bias, ACT_NONE, rowsum=True)
    ref = torch.stack([A[b].double() @ (B[b].double().t() if bt else B[b].double()) for b in range(batch)]) + bias.double()
    assert torch.equal(C, ref.to(TYPES[dtype]))
    # row sums of integers: exact while the sums of magnitudes stay below 2^24
    if float(ref.abs().sum(-1).max()) < 2 ** 24:
        assert torch.equal(rs.double(), ref.sum(-1))
    again, rs2 = call(_inside(A, offset), _inside(B, offset), bias, ACT_NONE, rowsum=True)
    assert torch.equal(C, again) and torch.equal(rs, rs2)


# `slices`: those of the 32 x 128 tiles on these shapes
@pytest.mark.parametrize("M,N,K,bt,slices", [(8, 4096, 8192, True, 16), (13, 4263, 8090, True, 15), (9, 4160, 7648, True, 14), (16, 4096, 4096, True, 8),
                                             (7, 5000, 4000, True, 7), (8, 5000, 5000, False, 9), (5, 11008, 4096, False, 6),
                                             (3, 12288, 8192, False, 6), (4, 13312, 16384, False, 5), (8, 4352, 2048, False, 4), (1, 1024, 1024, False, 2)])
def test_float32_sums_are_no_less_exact_than_in_slices(pgk, M, N, K, bt, slices):
    g = torch.Generator(device="cuda").manual_seed(K)
    A = torch.empty((1, M, K), device="cuda").uniform_(-1, 1, generator=g)
    B = torch.empty((1, N, K) if bt else (1, K, N), device="cuda").normal_(0, K ** -0.5, generator=g)
    ref = A[0].double() @ (B[0].double().t() if bt else B[0].double())

    def error(C):
        return float((C[0].double() - ref).norm() / ref.norm())
    one = error((pgk.gemm_fused_bt if bt else pgk.gemm_fused)(A, B, None, ACT_NONE, rowsum=False)[0])
    sliced = error((pgk.gemm_splitk_bt if bt else pgk.gemm_splitk)(A, B, None, ACT_NONE, splits=slices, rowsum=False)[0])
    # chains as long or shorter; the relative error of tens of thousands of such sums is the same to 1 %
    assert one <= 1.03 * sliced


@pytest.mark.parametrize("dtype,bt", [(F32, True), (F32, False), (BF16, True), (BF16, False)])
@pytest.mark.parametrize("act", [ACT_NONE, ACT_RELU, ACT_GELU_TANH, ACT_SILU])
def test_against_64_bits(pgk, dtype, bt, act):
    M, N, K = 13, 4230, 1016
    assert _one_pass(pgk, M, N, K, 1, dtype, bt)
    g = torch.Generator(device="cuda").manual_seed(act)
    A = torch.empty((1, M, K), device="cuda").uniform_(-1, 1, generator=g).to(TYPES[dtype])
    B = torch.empty((1, N, K) if bt else (1, K, N), device="cuda").normal_(0, K ** -0.5, generator=g).to(TYPES[dtype])
    bias = torch.empty(N, device="cuda").normal_(0, 0.1, generator=g)
    C, rs = (pgk.gemm_fused_bt if bt else pgk.gemm_fused)(A, B, bias, act, rowsum=True)
    x = A[0].double() @ (B[0].double().t() if bt else B[0].double()) + bias.double()
    ref = {ACT_NONE: lambda: x, ACT_RELU: lambda: x.clamp_min(0), ACT_SILU: lambda: x * torch.sigmoid(x),
           ACT_GELU_TANH: lambda: torch.nn.functional.gelu(x, approximate="tanh")}[act]()
    err = ((C[0].double() - ref).abs() / torch.maximum(ref.abs(), ref.pow(2).mean().sqrt())).max()
    # float32: sums of 1016 products in chains of at most 64 additions and the activation's few units; bf16: half a
    # unit of the stored result, 2^-9, and the sums
    assert err < (2.0 ** -16 if dtype == F32 else 2.0 ** -8)
    rs_err = (rs[0].double() - ref.sum(-1)).abs().max() / ref.abs().sum(-1).max()
    assert rs_err < 2.0 ** -18


def _integers(M, N, K, batch, dtype, seed=5):
    g = torch.Generator(device="cuda").manual_seed(seed)
    A = torch.randint(-7, 8, (batch, M, K), generator=g, device="cuda").to(TYPES[dtype])
    B = torch.randint(-7, 8, (batch, K, N), generator=g, device="cuda").to(TYPES[dtype])
    return A, B, torch.bmm(A.double(), B.double())


@pytest.mark.parametrize("dtype,M,N,K,bt", [(F32, 16, 2048, 64, False), (F32, 16, 2048, 128, True), (BF16, 16, 2048, 128, False), (BF16, 3, 600, 512, True)])
def test_a_workspace_for_the_tiles_row_sums_is_enough(pgk, dtype, M, N, K, bt):
    flags = pgk.WS_ROWSUM | (pgk.WS_B_TRANSPOSED if bt else 0)
    tiles = -(-(-(-N // 128)) * M * 4 // 256) * 256          # row sums per 128 columns
    assert _one_pass(pgk, M, N, K, 1, dtype, bt) and pgk.gemm_fused_workspace_bytes(M, N, K, 1, dtype, flags) > tiles
    A, B, ref = _integers(M, N, K, 1, dtype)
    call, B = (pgk.gemm_fused_bt, B.transpose(1, 2).contiguous()) if bt else (pgk.gemm_fused, B)
    ws = torch.full((tiles + 256,), 255, dtype=torch.uint8, device="cuda")
    C, rs = call(A, B, None, ACT_NONE, rowsum=True, workspace=ws[:tiles])
    assert torch.equal(C.double(), ref.to(TYPES[dtype]).double()) and torch.equal(rs.double(), ref.sum(-1))
    assert bool((ws[tiles:] == 255).all())
    with pytest.raises(pgk.PgkError):
        call(A, B, None, ACT_NONE, rowsum=True, workspace=ws[:tiles - 256])
