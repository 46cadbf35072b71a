"""fp32 products on the bf16 matrix cores (the 128 x 128 fp32 tile): values split into three bf16
terms, six products.  Compared element by element with the oracle under an a-priori bound, at the
step counts where the loop changes shape, on ragged edges, with both layouts of B, and on values
the terms cannot hold (the tile is then computed with the fp32 instruction)."""
import numpy as np
import pytest

from paper_2511_06345_amd import inputs as gen
from util import abs_inputs

pytestmark = pytest.mark.gpu
F32, NONE = gen.F32, gen.ACT_NONE


@pytest.fixture(scope="module")
def pgk():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2511_06345_amd import binding
    binding.load_library()
    return binding


def call(pgk, A, B, bt, splits=None):
    import torch
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(np.ascontiguousarray(np.swapaxes(B, 1, 2)) if bt else B).cuda()
    if splits is None:
        C, rs = pgk.gemm_fused(dA, dB, None, NONE, b_transposed=bt)
    else:
        C, rs = pgk.gemm_splitk(dA, dB, None, NONE, splits=splits, b_transposed=bt)
    torch.cuda.synchronize()
    return C.cpu().numpy(), rs.cpu().numpy()


def bound(K):
    """Largest error over sum |a||b| if every bf16 instruction (six per 32 k) cut the whole partial sum twice, by 2^-23
    each, and the products left out came to 2^-22.  The kernel rounds a whole partial sum twice per 32 k, to nearest,
    and leaves out 2^-24: this is what no result may miss, the tests of single kinds of data ask for more."""
    return (12 * -(-K // 32) + 2) * 2.0 ** -23


# (128 x 128 tiles: enough batch entries for 192 workgroups).  K: one step, its tail, two and three steps (the
# loop has none, then one in its middle), more, and their tails
SHAPES = [(128, 128, 32, 192), (128, 128, 5, 192), (130, 140, 64, 60), (129, 131, 70, 60), (200, 136, 96, 60), (128, 256, 224, 100),
          (256, 128, 256, 100), (250, 131, 259, 60), (128, 129, 288, 100), (131, 128, 516, 100)]


@pytest.mark.parametrize("bt", [False, True])
@pytest.mark.parametrize("shape", SHAPES)
def test_terms_meet_the_a_priori_bound(pgk, oracle, shape, bt):
    M, N, K, batch = shape
    assert pgk.gemm_plan(M, N, K, batch, F32, b_transposed=bt)["tile"] == (128, 128, 32)
    A = gen.normal(gen.tensor_seed(95, 1, M + K), batch * M * K, 1.0).reshape(batch, M, K)
    B = gen.normal(gen.tensor_seed(95, 2, N + K), batch * K * N, 1.0).reshape(batch, K, N)
    ref, ref_rs = oracle.gemm_fused(A, B, None, NONE)
    aa, ab, _ = abs_inputs(A, B, None, F32)
    scale, scale_rs = oracle.gemm_fused(aa, ab, None, NONE)
    for splits in (None, 2):
        if splits and K < 64:
            continue
        C, rs = call(pgk, A, B, bt, splits)
        assert np.all(np.abs(C - ref) <= bound(K) * scale), (shape, bt, splits)
        assert np.all(np.abs(rs - ref_rs) <= (bound(K) + N * 2.0 ** -23) * scale_rs), (shape, bt, splits)


@pytest.mark.parametrize("bt", [False, True])
def test_values_the_terms_cannot_hold(pgk, oracle, bt):
    """Infinities, NaNs, values above the largest bf16, rows and columns far below 2^-63 and down to
    denormals: as the fp32 instruction gives them, in their rows and columns and nowhere else."""
    M, N, K, batch = 256, 256, 288, 64
    A = gen.normal(gen.tensor_seed(96, 1), batch * M * K, 1.0).reshape(batch, M, K)
    B = gen.normal(gen.tensor_seed(96, 2), batch * K * N, 1.0).reshape(batch, K, N)
    A[1, 5, 7] = np.inf
    B[2, 11, 200] = -np.inf
    A[3, 130, 287] = np.nan
    A[4, 17, 9] = 3.4e38
    A[5, 20] *= np.float32(1e-30)
    A[6, 31] *= np.float32(1e-38)
    B[7, :, 3] *= np.float32(1e-42)
    A[8] *= np.float32(1e-33)
    B[8] *= np.float32(1e30)
    A[9, 40] = 0.0
    ref, _ = oracle.gemm_fused(A, B, None, NONE)
    aa, ab, _ = abs_inputs(A, B, None, F32)
    scale, _ = oracle.gemm_fused(aa, ab, None, NONE)
    C, _ = call(pgk, A, B, bt)
    with np.errstate(over="ignore"):
        want = ref.astype(np.float32)                   # (3.4e38 times more than one is an infinity in fp32)
    finite = np.isfinite(want)
    assert bool((np.isfinite(C) == finite).all()) and bool((np.isnan(C) == np.isnan(want)).all())
    assert bool((C[np.isinf(want)] == want[np.isinf(want)]).all())
    # (2^-149 per product: what fp32 sums of denormal products lose)
    assert np.all(np.abs(C - ref)[finite] <= (bound(K) * scale + K * 2.0 ** -149)[finite])
    assert np.all(C[9, 40] == 0.0)


def test_identity_is_exact_and_row_sums_have_no_bias(pgk):
    import torch
    n = 2048
    X = torch.empty((1, n, n), device="cuda").normal_(generator=torch.Generator("cuda").manual_seed(5))
    eye = torch.eye(n, device="cuda")[None].contiguous()
    assert torch.equal(pgk.gemm_fused(X, eye, None, NONE, rowsum=False)[0], X)
    assert torch.equal(pgk.gemm_fused(eye, X, None, NONE, rowsum=False)[0], X)
    # errors that are independent of each other weigh the same in a sum of outputs as in one output;
    # a common part of them would weigh sqrt(N) = 45 times as much
    W = torch.empty((1, n, n), device="cuda").normal_(generator=torch.Generator("cuda").manual_seed(6))
    C, rs = pgk.gemm_fused(X, W, None, NONE)
    ref = X[0].double() @ W[0].double()
    err = float((C[0].double() - ref).norm() / ref.norm())
    err_rs = float((rs[0].double() - ref.sum(1)).norm() / ref.sum(1).norm())
    err_cs = float((C[0].double().sum(0) - ref.sum(0)).norm() / ref.sum(0).norm())
    assert err < 2e-6 and err_rs < 2 * err and err_cs < 2 * err, (err, err_rs, err_cs)


def one_product_inputs(rows, cols, batch, seed):
    """A [batch][rows][64], B [batch][64][cols] of normal float32 values whose products have one term each: row m of A holds
    a value of 2^-60 ... 2^-122 at an even k, whose partners in B are as far above one, and a 1 beside it,
    whose partners are zero.  In odd entries the values of A have twelve significant bits (their low
    terms are denormal bf16 values and nothing is lost); odd rows are zero."""
    d = np.exp2(-60.0 - np.arange(64)).astype(np.float32)
    A, B = np.zeros((batch, rows, 64), np.float32), np.zeros((batch, 64, cols), np.float32)
    v = gen.normal(gen.tensor_seed(seed, 1, rows), batch * rows, 1.0).reshape(batch, rows)
    v[1::2] = (v[1::2].view(np.uint32) & np.uint32(0xfffff000)).view(np.float32)
    m = np.arange(0, rows, 2)
    A[:, m, m % 64] = v[:, m] * d[m % 64]
    A[:, m, m % 64 + 1] = 1.0
    B[:, ::2] = gen.normal(gen.tensor_seed(seed, 2, cols), batch * 32 * cols, 1.0).reshape(batch, 32, cols) / d[::2, None]
    return A, B


@pytest.mark.parametrize("bt", [False, True])
@pytest.mark.parametrize("small_b", [False, True])
@pytest.mark.parametrize("splits", [None, 2])
def test_small_values_beside_ordinary_ones(pgk, oracle, splits, small_b, bt):
    """Values whose low terms fall under the smallest bf16, in rows (columns) that hold ordinary values
    too, against values as far above one: nothing else in the sum hides what a term loses."""
    M, N, batch = 130, 140, 60
    assert pgk.gemm_plan(M, N, 64, batch, F32, b_transposed=bt)["tile"] == (128, 128, 32)
    if small_b:
        A, B = one_product_inputs(N, M, batch, 98)
        A, B = np.ascontiguousarray(np.swapaxes(B, 1, 2)), np.ascontiguousarray(np.swapaxes(A, 1, 2))
    else:
        A, B = one_product_inputs(M, N, batch, 98)
    ref, _ = oracle.gemm_fused(A, B, None, NONE)
    C, _ = call(pgk, A, B, bt, splits)
    assert np.all(np.abs(C - ref) <= bound(64) * np.abs(ref))


def test_small_values_in_a_convolution(pgk, oracle):
    import torch
    B, Cin, L, Cout = 8, 64, 4096, 130
    assert pgk.conv1d_workspace_bytes(B, Cin, L, Cout, 3, 1, 1, 1, F32) > 0
    wc, xc = one_product_inputs(Cout, L, B, 99)
    w = np.zeros((Cout, Cin, 3), np.float32)
    w[:, :, 1] = wc[0]
    y = pgk.conv1d(torch.from_numpy(xc).cuda(), torch.from_numpy(w).cuda(), None, NONE, 1, 1, 1).cpu().numpy()
    ref = oracle.conv1d(xc, w, None, NONE, 1, 1, 1)
    assert np.all(np.abs(y - ref) <= bound(3 * Cin) * np.abs(ref))


@pytest.mark.parametrize("power", [-66, -80, 60])
def test_scaling_by_a_power_of_two_changes_no_bit(pgk, power):
    """The terms hold values down to 2^-110 exactly: a factor of a power of two goes through the split, the
    products and the sums unchanged, so a result that differs in any bit took another route.  (Not for results
    below 2^-119, and of four million sums the smallest, by cancellation, is 2^-23 of an ordinary one: at a factor
    of 2^-80 that leaves 2^-100.)"""
    import torch
    g = torch.Generator("cuda").manual_seed(7)
    A = torch.randn((1, 1920, 200), generator=g, device="cuda")
    A = torch.where(A.abs() < 2.0 ** -8, torch.full_like(A, 0.5), A)
    B = torch.randn((1, 200, 2048), generator=g, device="cuda")
    assert pgk.gemm_plan(1920, 2048, 200, 1, F32)["tile"] == (128, 128, 32)
    C, _ = pgk.gemm_fused(A, B, None, NONE)
    D, _ = pgk.gemm_fused(A * 2.0 ** power, B, None, NONE)
    assert torch.equal(C * 2.0 ** power, D)


@pytest.mark.parametrize("bt", [False, True])
def test_results_near_the_smallest_normal_number(pgk, bt):
    """Factors the terms hold exactly, products of 2^-126 to 2^-108: their small parts fall under the smallest
    float32 inside the bf16 products."""
    import torch
    g = torch.Generator("cuda").manual_seed(8)
    n = 2048
    k = torch.arange(n, device="cuda")
    A = torch.diag(torch.rand(n, generator=g, device="cuda").add_(1.0) * torch.exp2(-63.0 + (k % 18)))[None].contiguous()
    B = torch.rand((1, n, n), generator=g, device="cuda").add_(1.0).mul_(2.0 ** -63)
    C, _ = pgk.gemm_fused(A, B.transpose(1, 2).contiguous() if bt else B, None, NONE, b_transposed=bt)
    ref = A[0].diagonal().double()[:, None] * B[0].double()
    assert bool(((C[0].double() - ref).abs() <= bound(32) / 12 * ref).all())


@pytest.mark.parametrize("value", [float("nan"), float("inf"), 1.25e-38, 3.4e38])
def test_columns_that_do_not_exist_leave_the_others_alone(pgk, value):
    """An odd row length: the last column is loaded together with the element after it, which belongs to
    the next row or the next batch entry.  Whatever that is, entry 0 gives the same bits."""
    import torch
    g = torch.Generator("cuda").manual_seed(9)
    M, N, K, batch = 256, 131, 70, 60
    assert pgk.gemm_plan(M, N, K, batch, F32)["tile"] == (128, 128, 32)
    A = torch.randn((batch, M, K), generator=g, device="cuda")
    B = torch.randn((batch, K, N), generator=g, device="cuda")
    C, rs = pgk.gemm_fused(A, B, None, NONE)
    B[1, 0, 0] = value
    D, rt = pgk.gemm_fused(A, B, None, NONE)
    assert torch.equal(C[0], D[0]) and torch.equal(rs[0], rt[0]) and torch.equal(C[2:], D[2:])


@pytest.mark.parametrize("pad", [0, 1])
def test_positions_that_do_not_exist_leave_the_others_alone(pgk, pad):
    """The same of a convolution: the last tile of a row reads on into the next row's input or its padding."""
    import torch
    g = torch.Generator("cuda").manual_seed(10)
    B, Cin, L, Cout = 8, 64, 4100, 128
    x = torch.randn((B, Cin, L), generator=g, device="cuda")
    w = torch.randn((Cout, Cin, 3), generator=g, device="cuda")
    y = pgk.conv1d(x, w, None, NONE, 1, pad, 1)
    x[1, :, 0] = float("nan")
    x[2, 5, 7] = 1.25e-38
    z = pgk.conv1d(x, w, None, NONE, 1, pad, 1)
    assert torch.equal(y[0], z[0]) and torch.equal(y[3:], z[3:])
    assert torch.equal(y[1:3, :, 128:], z[1:3, :, 128:])        # (all but the tiles that hold the two)


# how the values of A change along K (all of B: ordinary).  The rounding of a sum of K products is a random
# walk where errors are independent; where all are cut the same way, or a sum grows early, they add up
GROWTH = {"even": lambda t: np.ones_like(t), "rising": lambda t: np.exp2(20.0 * t - 20.0), "falling": lambda t: np.exp2(-20.0 * t),
          "early": lambda t: np.where(t < 0.25, 1.0, 2.0 ** -12), "middle": lambda t: np.where((t >= 0.25) & (t < 0.75), 64.0, 1.0)}


@pytest.mark.parametrize("K", [32, 224, 1024, 4096])
@pytest.mark.parametrize("growth", sorted(GROWTH))
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_sums_of_one_sign(pgk, sign, growth, K):
    """Per 32 k two roundings to nearest of a partial sum of at most the whole, 2^-24 / sqrt(3) each in the root
    mean square, independent of each other; within the 32, cuts of at most 2^-23 of their own sum.  And the errors of
    neighbouring outputs are independent: a sum over n of them has an error sqrt(n) times one's (three times that).
    (Not where most of a sum is there early: what then comes in pieces below half a unit of it is lost every time, in
    float32 sums of any order, and of a column's outputs in the same direction.)"""
    import torch
    n = 2048
    g = torch.Generator("cuda").manual_seed(K)
    A = torch.rand((1, n, K), generator=g, device="cuda") * torch.from_numpy(GROWTH[growth](np.arange(K) / K).astype(np.float32)).cuda()
    B = torch.rand((1, K, n), generator=g, device="cuda") * sign
    assert pgk.gemm_plan(n, n, K, 1, F32)["tile"] == (128, 128, 32)
    C, _ = pgk.gemm_fused(A, B, None, NONE)
    ref = A[0].double() @ B[0].double()
    err = (C[0].double() - ref) / ref.abs()
    each = 2.0 ** -24 * ((2 * -(-K // 32) / 3.0) ** 0.5 + 2.0)
    assert float(err.pow(2).mean().sqrt()) <= each
    if growth in ("early", "falling"):
        return
    assert float((C[0].double() - ref).sum(0).norm() / ref.sum(0).norm()) <= 3 * each / n ** 0.5
    assert float((C[0].double() - ref).sum(1).norm() / ref.sum(1).norm()) <= 3 * each / n ** 0.5


@pytest.mark.parametrize("bt", [False, True])
def test_one_product_per_output(pgk, bt):
    """A diagonal factor.  With x = h + m + l, |m| <= 2^-8 and |l| <= 2^-17 of x's power of two: the products left out are below
    2^-24 of a b (2 * 2^-25), the sum of the small ones is cut by less than 2^-27, and the last addition rounds to nearest."""
    import torch
    n = 2048
    g = torch.Generator("cuda").manual_seed(11)
    A = torch.diag(torch.randn(n, generator=g, device="cuda"))[None].contiguous()
    B = torch.randn((1, n, n), generator=g, device="cuda")
    C, _ = pgk.gemm_fused(A, B.transpose(1, 2).contiguous() if bt else B, None, NONE, b_transposed=bt)
    ref = A[0].diagonal().double()[:, None] * B[0].double()
    err = (C[0].double() - ref).abs() / ref.abs()
    assert float(err.max()) <= 2.25 * 2.0 ** -24
    # rounding to nearest alone: 0.42 ... 0.43 of 2^-24 for values spread over a power of two
    assert float(err.pow(2).mean().sqrt()) <= 0.46 * 2.0 ** -24
