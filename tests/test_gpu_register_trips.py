"""bf16 products and convolutions whose tiles are copied through registers: every number of K tiles around the main loop's trips of
two and its end, the last tile whole and not.  Small integers: sums exact in float32, rounded once."""
import pytest
import torch

from paper_2511_06345_amd import binding as pgk

gpu = pytest.mark.gpu


def test_longer_sums_go_through_registers():
    """Odd rows on both sides of the choice: no workspace but for partial products where they are not copied first."""
    def copied(M, N, K, bt):
        slices = pgk.gemm_plan(M, N, K, 1, 1, bt)["slices"]
        partials = 0 if slices == 1 else -(-slices * M * N * 4 // 256) * 256
        return pgk.gemm_fused_workspace_bytes(M, N, K, 1, 1, pgk.WS_B_TRANSPOSED if bt else 0) != partials

    assert not copied(435, 37339, 429, True)         # 73 us copied, 56 through registers
    assert not copied(7616, 53, 1225, False)         # 37 / 26
    assert copied(4096, 4095, 4095, False)           # 126 / 180


@gpu
@pytest.mark.parametrize("tiles", range(1, 11))
@pytest.mark.parametrize("M,N,bt", [(500, 20001, False), (1000, 2303, False), (1000, 2303, True), (40, 130, True)])
def test_products(tiles, M, N, bt):
    for K in (64 * tiles, 64 * tiles - 1, 64 * tiles - 63):
        g = torch.Generator(device="cuda").manual_seed(K)
        A = torch.randint(-7, 8, (1, M, K), generator=g, device="cuda").bfloat16()
        B = torch.randint(-7, 8, (1, N, K) if bt else (1, K, N), generator=g, device="cuda").bfloat16()
        C = pgk.gemm_fused(A, B, None, 0, b_transposed=bt)[0]
        ref = A[0].double() @ (B[0].t() if bt else B[0]).contiguous().double()
        assert torch.equal(C.view(M, N), ref.float().bfloat16()), K


@gpu
@pytest.mark.parametrize("blocks,Kw", [(1, 1), (1, 3), (2, 2), (1, 5), (2, 3), (1, 7), (4, 2), (3, 3)])
@pytest.mark.parametrize("Cout,L", [(40, 5001), (100, 3001), (300, 4001)])
def test_convolutions(blocks, Kw, Cout, L):
    g = torch.Generator(device="cuda").manual_seed(Kw)
    x = torch.randint(-3, 4, (4, 64 * blocks, L), generator=g, device="cuda").bfloat16()
    w = torch.randint(-3, 4, (Cout, 64 * blocks, Kw), generator=g, device="cuda").bfloat16()
    y = pgk.conv1d(x, w, None, 0, 1, 1, 1)
    xp = torch.nn.functional.pad(x.double(), (1, 1))
    ref = torch.stack([sum(w[:, :, k].double() @ xp[b, :, k:k + y.shape[2]].contiguous() for k in range(Kw)) for b in range(4)])
    assert torch.equal(y, ref.float().bfloat16())
