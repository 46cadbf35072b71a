"""The second passes that add K slices and row-sum partials, at the remainders of their load batches.

The operands are small whole numbers: every product and partial sum is exact in float32, so a slice or a
partial that is left out, read twice or read from elsewhere changes the result, and the tolerance is 0.
"""
import pytest
import torch

import paper_2511_06345_amd as pgk

pytestmark = pytest.mark.gpu


def _ints(shape, seed, dtype):
    g = torch.Generator().manual_seed(seed)
    return torch.randint(-3, 4, shape, generator=g).to(dtype)


def _check(A, B, bias, C, rs):
    # |sum| <= 9 * K < 2^24 in C, and the row sums stay below 2^24 for the drawn operands
    ref = A.double() @ B.double() + bias.double()
    assert float(ref.abs().sum(-1).max()) < 2 ** 24
    assert torch.equal(C.double().cpu(), ref)
    assert torch.equal(rs.double().cpu(), ref.sum(-1))


@pytest.mark.parametrize("splits", [2, 3, 4, 5, 7, 8, 9, 10, 16])
@pytest.mark.parametrize("N", [300, 301])       # four columns a lane, and one
def test_slices(splits, N):
    M, K = 5, 64 * splits
    A, B, bias = _ints((1, M, K), 1, torch.float32), _ints((1, K, N), 2, torch.float32), _ints((N,), 3, torch.float32)
    C, rs = pgk.gemm_splitk(A.cuda(), B.cuda(), bias.cuda(), 0, splits=splits)
    _check(A, B, bias, C, rs)


@pytest.mark.parametrize("tiles", [1, 2, 4, 8, 9, 12, 16, 17, 18, 32, 33, 48])
def test_row_sum_partials(tiles):
    M, N, K = 512, 64 * tiles, 128
    A, B, bias = _ints((1, M, K), 4, torch.float32), _ints((1, K, N), 5, torch.float32), _ints((N,), 6, torch.float32)
    C, rs = pgk.gemm_fused(A.cuda(), B.cuda(), bias.cuda(), 0)
    _check(A, B, bias, C, rs)


def test_row_sum_partials_that_are_not_finite():
    M, N, K = 70, 640, 128
    A, B = _ints((1, M, K), 7, torch.float32).cuda(), _ints((1, K, N), 8, torch.float32).cuda()
    inf = float("inf")
    for places, want in (({3: inf}, inf), ({600: -inf}, -inf), ({3: inf, 600: -inf}, float("nan")), ({100: float("nan")}, float("nan")),
                         ({3: 3e38, 600: 3e38}, inf), ({3: 3e38, 300: 3e38, 600: -inf}, -inf)):
        bias = torch.zeros(N)
        for n, v in places.items():
            bias[n] = v
        rs = pgk.gemm_fused(A, B, bias.cuda(), 0)[1].cpu()
        assert torch.equal(torch.full_like(rs, want).isnan(), rs.isnan()) and (want != want or bool((rs == want).all())), (places, rs)


@pytest.mark.parametrize("dtype,bt", [(torch.float32, False), (torch.bfloat16, True)])
def test_row_sums_of_many_tile_columns_are_rounded_once(dtype, bt):
    # non-negative whole numbers: sums inside a tile stay below 2^24 and are exact, those of a row do not, and the partials are
    # added in 64 bits, exactly, so the result is the exact sum rounded once
    M, N, K = 512, 64 * 301, 255
    g = torch.Generator().manual_seed(9)
    A = torch.randint(0, 8, (1, M, K), generator=g).to(dtype).cuda()
    B = torch.randint(0, 8, (1, N, K) if bt else (1, K, N), generator=g).to(dtype).cuda()
    rs = (pgk.gemm_fused_bt if bt else pgk.gemm_fused)(A, B, None, 0)[1]
    ref = (A[0].double() @ (B[0].double().t() if bt else B[0].double())).sum(-1)
    assert float(ref.min()) > 2 ** 24
    assert torch.equal(rs[0], ref.float())
