"""Unsplit fp32 products whose last round of 128 x 128 tiles does a good part of a round: they run on that
tile, up to a quarter of a round on the 64 x 64 one.  Both sides of the line, in the forms that the calls take."""
import pytest
import torch

from paper_2511_06345_amd import binding as pgk

gpu = pytest.mark.gpu
LARGE, SMALL = (128, 128, 32), (64, 64, 32)
# last rounds of 64 and 65 workgroups, of a whole round (512), ragged M, N and K, narrow, batched
CASES = [((2048, 2560, 1024, 1), SMALL), ((384, 13696, 1024, 1), LARGE), ((2801, 2000, 1030, 1), LARGE),
         ((4096, 2048, 1028, 1), LARGE), ((130, 30001, 1025, 1), LARGE), ((300, 700, 1030, 25), LARGE)]


@pytest.mark.parametrize("bt", [False, True])
@pytest.mark.parametrize("shape, tile", CASES)
def test_choice(shape, tile, bt):
    assert pgk.gemm_plan(*shape, 0, b_transposed=bt)["tile"] == tile


@gpu
@pytest.mark.parametrize("bt", [False, True])
@pytest.mark.parametrize("shift", [0, 1])       # elements that A starts off a 16-byte boundary
@pytest.mark.parametrize("shape, tile", CASES)
def test_values(shape, tile, shift, bt):
    M, N, K, batch = shape
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    A = torch.randn(batch * M * K + shift, generator=g, device="cuda")[shift:].view(batch, M, K)
    B = torch.randn(batch, *((N, K) if bt else (K, N)), generator=g, device="cuda")
    C, rs = pgk.gemm_fused(A, B, None, 0, b_transposed=bt)
    # a sum of K products in float32: at most K roundings of 2^-24 of sum |a||b| (the fp32 instruction; in bf16
    # terms two per 32 k and a few at the size of 32 products); the row sums add N more roundings
    per_sum = (K + 2) * 2.0 ** -24
    for b in range(batch):
        a, w = A[b].double(), (B[b].t() if bt else B[b]).contiguous().double()
        ref, scale = a @ w, a.abs() @ w.abs()
        assert bool(((C[b].double() - ref).abs() <= per_sum * scale).all())
        assert bool(((rs[b].double() - ref.sum(-1)).abs() <= (per_sum + N * 2.0 ** -24) * scale.sum(-1)).all())
