"""bf16 products and convolutions whose tiles are copied through registers: every number of K tiles around the main loop's trips of
two and its end, for products the last tile whole and not.  Small integers: sums exact in float32, rounded once."""
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


# tile, K tiles: B, Cin, L, Cout, Kw, pad, dilation, elements that x starts past a 16-byte boundary; sizes that the planner sends to each tile
# that copies a convolution's input through registers (test_kernels_reached_cpu.py asserts it)
CONVOLUTIONS = {
    (128, 128, 2): (116, 128, 60, 512, 1, 0, 1, 1), (128, 128, 3): (78, 192, 130, 102, 1, 0, 3, 1), (128, 128, 4): (1, 256, 68, 96, 1, 0, 1, 1),
    (128, 128, 5): (1, 320, 79, 43, 1, 0, 3, 0), (128, 128, 6): (1, 384, 82, 43, 1, 0, 1, 1), (128, 128, 7): (1, 448, 84, 65, 1, 0, 1, 1),
    (128, 128, 8): (2, 512, 66, 57, 1, 0, 3, 1), (128, 128, 9): (37, 192, 135, 384, 3, 3, 3, 0), (128, 128, 10): (12, 320, 181, 34, 2, 1, 1, 0),
    (128, 256, 2): (42, 128, 1372, 69, 1, 0, 1, 1), (128, 256, 3): (14, 192, 3871, 72, 1, 0, 1, 0), (128, 256, 4): (128, 128, 269, 73, 2, 0, 1, 0),
    (128, 256, 5): (98, 320, 270, 96, 1, 0, 1, 1), (128, 256, 6): (96, 384, 300, 96, 1, 0, 1, 1), (128, 256, 7): (101, 448, 257, 96, 1, 0, 1, 0),
    (128, 256, 8): (117, 256, 295, 68, 2, 0, 1, 0), (128, 256, 9): (52, 192, 927, 77, 3, 0, 3, 0), (128, 256, 10): (118, 320, 259, 96, 2, 1, 3, 0),
    (256, 128, 2): (50, 128, 74, 1000, 1, 1, 3, 0), (256, 128, 3): (49, 192, 67, 1000, 1, 0, 1, 0), (256, 128, 4): (115, 256, 67, 384, 1, 0, 1, 0),
    (256, 128, 5): (118, 320, 68, 384, 1, 0, 1, 1), (256, 128, 6): (101, 384, 97, 384, 1, 0, 1, 0), (256, 128, 7): (127, 448, 64, 324, 1, 1, 1, 0),
    (256, 128, 8): (100, 256, 66, 384, 2, 0, 1, 0), (256, 128, 9): (102, 192, 97, 384, 3, 3, 3, 0), (256, 128, 10): (103, 320, 103, 384, 2, 0, 1, 0),
    (256, 256, 1): (121, 64, 428, 256, 1, 1, 3, 0), (256, 256, 2): (96, 128, 146, 512, 1, 0, 1, 1), (256, 256, 3): (46, 192, 139, 1000, 1, 1, 1, 0),
    (256, 256, 4): (68, 128, 652, 129, 2, 0, 1, 0), (256, 256, 5): (34, 320, 134, 1000, 1, 0, 1, 1), (256, 256, 6): (12, 384, 2958, 137, 1, 0, 3, 1),
    (256, 256, 7): (43, 448, 154, 670, 1, 0, 1, 1), (256, 256, 8): (143, 256, 143, 162, 2, 0, 1, 0), (256, 256, 9): (102, 192, 136, 384, 3, 3, 3, 0),
    (256, 256, 10): (68, 320, 151, 395, 2, 0, 1, 0), (256, 256, 24): (8, 512, 4096, 512, 3, 1, 1, 0),
}


@gpu
@pytest.mark.parametrize("tile", CONVOLUTIONS)
def test_convolutions_by_tile(tile):
    B, Cin, L, Cout, Kw, pad, dilation, off = CONVOLUTIONS[tile]
    g = torch.Generator(device="cuda").manual_seed(L)
    x = torch.randint(-3, 4, (B * Cin * L + off,), generator=g, device="cuda").bfloat16()[off:].view(B, Cin, L)
    w = torch.randint(-3, 4, (Cout, Cin, Kw), generator=g, device="cuda").bfloat16()
    bias = torch.randint(-7, 8, (Cout,), generator=g, device="cuda").float()
    y = pgk.conv1d(x, w, bias, 0, 1, pad, dilation)
    for b in range(B):
        xp = torch.nn.functional.pad(x[b].double(), (pad, pad))
        ref = sum(w[:, :, k].double().contiguous() @ xp[:, k * dilation:k * dilation + y.shape[2]].contiguous() for k in range(Kw)) + bias.double()[:, None]
        assert torch.equal(y[b], ref.float().bfloat16()), b


@gpu
def test_convolution_without_room_for_copies_goes_through_registers():
    """Copies of the input are the faster way here; a workspace that holds the regrouped weights and the rows' ends is enough all the same."""
    B, Cin, L, Cout, Kw = WITHOUT_ROOM
    need = pgk.conv1d_workspace_least_bytes(B, Cin, L, Cout, Kw, 1, 0, 1, 1)
    g = torch.Generator(device="cuda").manual_seed(8)
    x = torch.randint(-3, 4, (B, Cin, L), generator=g, device="cuda").bfloat16()
    w = torch.randint(-3, 4, (Cout, Cin, Kw), generator=g, device="cuda").bfloat16()
    ws = torch.full((need,), 255, dtype=torch.uint8, device="cuda")
    y = pgk.conv1d(x, w, None, 0, workspace=ws[:need // 2 // 256 * 256])
    ref = sum(w[:, :, k].double().contiguous() @ x[0, :, k:k + y.shape[2]].double() for k in range(Kw))
    assert torch.equal(y[0], ref.float().bfloat16()) and torch.equal(y, pgk.conv1d(x, w, None, 0))
    assert bool((ws[need // 2:] == 255).all())


WITHOUT_ROOM = (1, 256, 190, 39, 2)
