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


@pytest.mark.parametrize("tiles", [1, 2, 4, 8, 9, 12, 16, 17])
def test_row_sum_partials(tiles):
    M, N, K = 512, 64 * tiles, 128
    A, B, bias = _ints((1, M, K), 4, torch.float32), _ints((1, K, N), 5, torch.float32), _ints((N,), 6, torch.float32)
    C, rs = pgk.gemm_fused(A.cuda(), B.cuda(), bias.cuda(), 0)
    _check(A, B, bias, C, rs)
