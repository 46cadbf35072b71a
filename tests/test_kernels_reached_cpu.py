"""The kernels behind the dispatch (no GPU: tests/launches.py): which one a size goes to where two were measured, and that the sizes of
the GPU tests reach the kernels they are meant for."""
import pytest

import test_gpu_conv_bf16_in_place as in_place
import test_gpu_conv_in_place as in_place_fp32
import test_gpu_reduce_block as blocks
import test_gpu_register_trips as trips
from launches import traced
from paper_2511_06345_amd import inputs as gen

F32, BF16 = gen.F32, gen.BF16


def first_kernels(calls, **how):
    return [call if isinstance(call, int) else call[0].kernel for call in traced(calls, **how)]


# us in the kernels with lanes along the inner dimension / with a workgroup per block
BLOCK_OR_LANES = [
    (F32, (5, 8632, 7), 7.2, 12.4), (F32, (11, 1969, 13), 7.3, 10.2), (F32, (77, 2865, 3), 8.9, 7.4), (BF16, (249, 461, 63), 21.4, 9.1),
    (BF16, (9, 585, 199), 8.0, 11.8), (BF16, (261, 55, 285), 6.1, 13.4), (BF16, (446, 21, 87), 4.6, 8.6), (F32, (164, 52, 339), 5.4, 8.1),
    (F32, (5299, 342, 7), 14.1, 24.8), (F32, (1436, 3222, 3), 1.37, 1.0), (F32, (7361, 20, 207), 25.4, 38.5), (BF16, (976, 21, 25), 0.67, 1.0),
    (BF16, (570, 830, 2), 1.52, 1.0), (BF16, (303, 861, 873), 92.9, 123.8), (BF16, (29, 22832, 138), 2.12, 1.0), (F32, (14, 2533, 47), 0.81, 1.0),
    (F32, (178, 3508, 25), 1.62, 1.0), (BF16, (1, 39012, 5), 9.2, 27.5), (F32, (28, 49714, 67), 1.91, 1.0), (BF16, (5, 4283, 282), 11.1, 14.5),
]


def test_blocks_where_they_are_faster():
    kernels = first_kernels([("reduce_max", dtype, *shape) for dtype, shape, _, _ in BLOCK_OR_LANES])
    for (dtype, shape, lanes, block), kernel in zip(BLOCK_OR_LANES, kernels):
        assert kernel.startswith("reduce_max_block_kernel") == (block < lanes), (dtype, shape, kernel)


def test_long_fp32_rows_in_the_faster_workgroup():
    """us at 600 MB with 512 threads / 1024: 12288 elements 89.3 / 87.5, 16384 94 / 89, 20480 89 / 88; 16448 93 / 95, 28672 90.6 / 91.2; 512 for bf16."""
    rows = [(F32, 12288, 1024), (F32, 16384, 1024), (F32, 20480, 1024), (F32, 16448, 512), (F32, 28672, 512), (F32, 8448, 512), (BF16, 32768, 512)]
    for (dtype, red, threads), (launch,) in zip(rows, traced([("reduce_max", dtype, 150000000 // red, red, 1) for dtype, red, _ in rows])):
        assert launch.kernel.startswith("reduce_max_held_rows_kernel") and launch.block == threads, (dtype, red, launch)


@pytest.mark.parametrize("dtype", [F32, BF16])
def test_sizes_for_the_block_kernel_reach_it(dtype):
    name = "reduce_max_block_kernel<%s, " % ("true" if dtype == BF16 else "false")
    for R, outer, inner in blocks.EDGES[dtype]:
        calls = [("reduce_max", dtype, outer, red, inner) for red in blocks.edges(dtype, R, outer, inner)]
        for off in (0, 1):
            reached = [kernel == name + ("256>" if outer == 520 else "1024>") for kernel in first_kernels(calls, x_off=off)]
            assert all(reached) if off == 0 else sum(reached) >= 4, (off, list(zip(calls, reached)))
    in_segments = [len(call) == 2 for call in traced([("reduce_max", dtype, *shape) for shape in blocks.SHAPES]) if call[0].kernel == name + "256>"]
    assert in_segments.count(True) >= 2 and in_segments.count(False) >= 2


def test_short_fp32_sums_are_plain_multiply_adds():
    """Convolutions with fewer than 12 products per output stay off the kernel of three terms, which rounds a single product worse."""
    calls = [("conv1d", F32, B, Cin, L, Cout, Kw, stride, 1, 1) for Cin, Kw in ((1, 1), (2, 1), (1, 3), (5, 1), (2, 5), (11, 1), (12, 1), (4, 3), (16, 1))
             for B, L, Cout, stride in ((1, 300, 40, 1), (3, 5000, 33, 2), (2, 20000, 200, 1))]
    for call, kernel in zip(calls, first_kernels(calls)):
        if call[3] * call[6] < 12:
            assert "f32_terms" not in kernel, (call, kernel)
    assert any("f32_terms" in kernel for kernel in first_kernels(calls[-9:]))


def test_convolutions_in_place_take_no_more_workspace_than_they_write_to():
    """fp32 none, bf16 the regrouped weights, though the views of such sizes would take copies of the input; with less the call is refused
    where the views are another way, and the views take what they took."""
    from paper_2511_06345_amd import binding
    fp32, bf16 = (F32, 10, 152, 53120, 19, 7, 1, 0, 1), (BF16, 13, 384, 11631, 61, 5, 2, 0, 1)
    assert binding.conv1d_workspace_bytes(*fp32[1:], F32) > 300e6 and binding.conv1d_workspace_least_bytes(*fp32[1:], F32) == 0
    least = binding.conv1d_workspace_least_bytes(*bf16[1:], BF16)
    assert binding.conv1d_workspace_bytes(*bf16[1:], BF16) > 200e6 and 61 * 384 * 5 * 2 <= least < 61 * 384 * 5 * 2 + 256
    for call, room in ((fp32, 0), (bf16, least)):
        (with_all,), (with_least,) = traced([("conv1d", *call)]), traced([("conv1d", *call)], workspace=room)
        assert with_all == with_least and ("f32_terms" in with_all[-1].kernel or "conv_bf16" in with_all[-1].kernel), (with_all, with_least)
    assert traced([("conv1d", *bf16)], workspace=least - 256) == [-3]
    views = (F32, 2, 64, 1024, 32, 3, 1, 1, 1)
    assert binding.conv1d_workspace_bytes(*views[1:], F32) == binding.conv1d_workspace_least_bytes(*views[1:], F32) > 0
    assert traced([("conv1d", *views)], workspace=0) == [-3]


def last_kernels(calls, **how):
    return [call if isinstance(call, int) else call[-1].kernel for call in traced(calls, **how)]


def test_sizes_for_each_instance_of_the_bf16_convolution_reach_it():
    for off in (0, 1):
        kernels = last_kernels([("conv1d", BF16, *case) for _, case in in_place.INSTANCES], x_off=off)
        for ((rows, groups, parts), case), kernel in zip(in_place.INSTANCES, kernels):
            assert kernel == f"conv_bf16_kernel<{rows}, {groups}, {str(parts).lower()}>", (case, kernel)
    reached = {instance for instance, _ in in_place.INSTANCES}
    assert reached == {(rows, groups, parts) for rows in (32, 64, 128) for groups in (1, 2, 3) for parts in (False, True)} - {(r, 1, True) for r in (32, 64, 128)}
    # with one workgroup, rows of two elements, 384 positions
    alone = traced([("conv1d", BF16, *case) for instance, case in in_place.INSTANCES if case[0] == 1])
    assert sum(call[-1].grid == 1 for call in alone) >= 6
    assert any((case[4] - 1) * case[7] + 127 * case[5] + 1 == 384 for _, case in in_place.INSTANCES) and any(case[2] == 2 for _, case in in_place.INSTANCES)


def test_sizes_for_each_tile_through_registers_reach_it():
    for off in (0, 1):
        sizes = [(tile, case) for tile, case in trips.CONVOLUTIONS.items() if case[-1] == off]
        kernels = last_kernels([("conv1d", BF16, B, Cin, L, Cout, Kw, 1, pad, dil) for _, (B, Cin, L, Cout, Kw, pad, dil, _) in sizes], x_off=off)
        for (((rows, cols, tiles), case), kernel) in zip(sizes, kernels):
            assert kernel.startswith(f"gemm_mfma_kernel<MfmaCfgReg<false, {rows}, {cols}, 64") and case[1] // 64 * case[4] == tiles, (case, kernel)
    from paper_2511_06345_amd import binding
    B, Cin, L, Cout, Kw = trips.WITHOUT_ROOM
    need = binding.conv1d_workspace_least_bytes(B, Cin, L, Cout, Kw, 1, 0, 1, BF16)
    copies, registers = last_kernels([("conv1d", BF16, B, Cin, L, Cout, Kw, 1, 0, 1)] * 2, workspace=[need, need // 2 // 256 * 256])
    assert "MfmaCfg<" in copies and "MfmaCfgReg<" in registers


def test_sizes_for_the_fp32_convolution_in_place_reach_each_tile():
    for off in (0, 1):
        kernels = last_kernels([("conv1d", F32, *case) for case in in_place_fp32.CASES], x_off=off)
        steps = {}
        for case, kernel in zip(in_place_fp32.CASES, kernels):
            steps.setdefault(kernel, set()).add(-(-case[1] * case[4] // 32))
        for rows in (128, 64, 32):
            reached = [n for kernel, n in steps.items() if kernel.startswith(f"conv_f32_terms_kernel<TermsCfg<false, {rows}, 128")]
            assert reached and len(reached[0]) >= 3, (rows, steps)


# us in the views or copies of the input / in place
VIEWS_OR_IN_PLACE = [
    (F32, (1, 256, 131200, 19, 10, 2, 0, 1), 162, 229), (F32, (3, 767, 6239, 512, 3, 4, 0, 1), 148, 261), (F32, (22, 256, 3515, 1, 10, 2, 0, 3), 107, 156),
    (F32, (9, 95, 8505, 16, 10, 2, 0, 1), 47, 61), (F32, (10, 152, 53120, 19, 7, 1, 0, 1), 450, 305), (F32, (16, 57, 36868, 67, 5, 1, 0, 1), 314, 246),
    (F32, (2, 463, 2816, 24, 5, 1, 0, 1), 51, 82), (BF16, (2, 665, 11631, 392, 10, 2, 4, 1), 113, 180), (BF16, (1, 256, 16069, 557, 7, 2, 3, 1), 40, 58),
    (BF16, (19, 512, 836, 256, 7, 1, 3, 1), 66, 79), (BF16, (27, 275, 1422, 233, 10, 2, 36, 8), 55, 72), (BF16, (13, 384, 11631, 61, 5, 2, 0, 1), 117, 58),
    (BF16, (13, 64, 4673, 128, 7, 2, 0, 1), 39, 17), (BF16, (8, 512, 4096, 512, 3, 1, 1, 1), 56, 86), (BF16, (13, 17, 61760, 64, 1, 1, 0, 1), 85, 27),
]


def test_convolutions_in_place_where_that_is_faster():
    kernels = last_kernels([("conv1d", dtype, *case) for dtype, case, _, _ in VIEWS_OR_IN_PLACE])
    for (dtype, case, views, in_place_us), kernel in zip(VIEWS_OR_IN_PLACE, kernels):
        assert kernel.startswith(("conv_f32_terms", "conv_bf16")) == (in_place_us < views), (dtype, case, kernel)


def test_strided_reductions_with_little_workspace():
    """Where the faster way needs segments and there is no room for them, whole blocks in one launch, or in fewer segments; refused where those
    do not fit either."""
    from paper_2511_06345_amd import binding
    blocks_in_one = [(F32, 5, 8632, 7), (F32, 11, 1969, 13), (BF16, 9, 585, 199), (BF16, 4, 2000, 64)]
    for call, full, (launch,) in zip(blocks_in_one, traced([("reduce_max", *c) for c in blocks_in_one]), traced([("reduce_max", *c) for c in blocks_in_one], workspace=0)):
        assert binding.reduce_max_workspace_bytes(*call[1:], call[0]) > 0 and len(full) == 2 and "block" not in full[0].kernel
        assert launch.kernel.startswith("reduce_max_block_kernel") and launch.block == 1024
    # [4, 9811, 14]: 298 segments the faster way, 34 of whole blocks
    few = ("reduce_max", F32, 4, 9811, 14)
    enough = 34 * 4 * 14 * 8
    assert binding.reduce_max_workspace_bytes(*few[2:], F32) > enough
    segments, refused = traced([few, few], workspace=[enough, enough - 8])
    assert segments[0].kernel.startswith("reduce_max_block_kernel") and len(segments) == 2 and refused == -3
    assert traced([("reduce_max", BF16, 128, 24742, 88), ("reduce_max", F32, 16, 1 << 24, 1)], workspace=0) == [-3, -3]
