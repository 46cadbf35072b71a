"""Max reduction over a strided dimension by workgroups that sweep whole blocks (inner extents up to about
half of what a workgroup loads at once): exact against the oracle, values and first positions, at the edges of periods,
batches of periods, segments and blocks, for starts of X on and off the 16-byte grid."""
import numpy as np
import pytest

from paper_2511_06345_amd import inputs as gen
from test_gpu_reduce_unaligned import check

pytestmark = pytest.mark.gpu
F32, BF16 = gen.F32, gen.BF16


@pytest.fixture(scope="module")
def pgk():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2511_06345_amd import binding
    binding.load_library()
    return binding


# r per period of 1024 threads (one launch): bf16 7 -> 1168, 250 -> 32; fp32 7 -> 584, 250 -> 16
PERIODS = {BF16: (1168, 32), F32: (584, 16)}
SHAPES = [(3, 700, 9), (1, 30000, 2), (2, 64, 1500), (2, 70, 2047), (5, 40, 100),      # one launch
          (3, 90000, 5), (5, 40000, 33), (2, 60001, 64), (7, 20000, 71), (300, 3000, 25),      # segments
          (600, 333, 21), (1100, 701, 13), (520, 90, 250), (1030, 4, 1000)]             # a workgroup per outer index


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("shape", SHAPES)
def test_blocks(pgk, oracle, dtype, shape):
    n = shape[0] * shape[1] * shape[2]
    x = gen.uniform(gen.tensor_seed(99, 1, n), n, -1.0, 1.0)
    x = (gen.f32_to_bf16_bits(x) if dtype == BF16 else x).reshape(shape)
    for start in (0, 1, 2, 3):
        check(pgk, oracle, x, start, dtype)


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("inner", [7, 250])
def test_edges_of_periods(pgk, oracle, dtype, inner):
    R = PERIODS[dtype][inner == 250]
    for red in (R - 1, R, R + 1, 2 * R, 4 * R - 1, 4 * R, 4 * R + 1, 5 * R, 8 * R + 1, 9 * R):
        if red * inner * (2 if dtype == BF16 else 4) > 256 << 10:
            continue
        x = gen.small_ints(gen.tensor_seed(99, 2, red), 2 * red * inner, -2, 2).reshape(2, red, inner)
        x[0] = 0.0
        x[0, np.arange(inner) % red, np.arange(inner)] = 1.0          # one maximum per column, in every lane's reach
        x[0, red - 1, inner - 1] = 2.0
        for start in (0, 1, 3):
            check(pgk, oracle, gen.f32_to_bf16_bits(x) if dtype == BF16 else x, start, dtype)


# edges of periods, batches of periods and blocks on the block kernel itself (test_kernels_reached_cpu.py): blocks enough for 1024 threads each
# instead of two launches, and a workgroup of 256 each (r per period, then outer and inner)
EDGES = {F32: [(584, 200, 7), (100, 200, 40), (40, 200, 100), (144, 520, 7), (28, 520, 36)],
         BF16: [(1168, 200, 7), (204, 100, 40), (32, 100, 250), (288, 520, 7), (56, 520, 36)]}


def edges(dtype, R, outer, inner):
    """Those of the edges where the block kernel is the one that runs."""
    es = 2 if dtype == BF16 else 4
    least = (7400 if dtype == F32 else 2048) if outer == 520 else 64 * es * inner if inner >= 100 else 0
    return [red for red in (R - 1, R, R + 1, 2 * R, 4 * R - 1, 4 * R, 4 * R + 1, 5 * R, 8 * R + 1, 9 * R) if red * inner * es >= least]


@pytest.mark.parametrize("dtype,R,outer,inner", [(dtype, *e) for dtype in (F32, BF16) for e in EDGES[dtype]])
def test_edges_of_periods_in_many_blocks(pgk, oracle, dtype, R, outer, inner):
    reds = edges(dtype, R, outer, inner)
    assert len(reds) >= 4
    for red in reds:
        x = gen.small_ints(gen.tensor_seed(99, 4, red), outer * red * inner, -2, 2).reshape(outer, red, inner)
        x[:2] = 0.0
        x[:2, np.arange(inner) % red, np.arange(inner)] = 1.0
        x[0, red - 1, inner - 1] = 2.0
        for start in (0, 1, 3):
            check(pgk, oracle, gen.f32_to_bf16_bits(x) if dtype == BF16 else x, start, dtype)


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("shape", [(4, 3000, 6), (3, 50000, 11), (2, 30011, 65), (530, 200, 33), (60, 400, 9), (12, 17003, 65)])
def test_special_values(pgk, oracle, dtype, shape):
    """Slices of nothing but -inf, signed zeros, maxima and NaNs in the first and last places."""
    outer, red, inner = shape
    x = gen.uniform(gen.tensor_seed(99, 3), outer * red * inner, -1.0, 0.5).reshape(shape)
    x[0, :, 0] = -np.inf
    x[0, :, 1] = -np.inf
    x[0, red - 1, 1] = -1e30
    x[0, 1, 2], x[0, red - 2, 2] = np.nan, 3.0
    x[0, red - 1, 3] = np.nan
    x[0, :, 4] = -0.0
    x[0, 5:, 4] = 0.0
    x[0, :, 5] = np.nan
    x[1, 0], x[1, red - 1] = 2.0, 2.0
    x[-1, red - 1] = 4.0
    x[-1, 0, inner - 1] = np.nan
    x = gen.f32_to_bf16_bits(x) if dtype == BF16 else x
    for start in (0, 1, 3):
        check(pgk, oracle, x, start, dtype)


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("shape", [(5, 8632, 7), (11, 1969, 13), (9, 320, 199), (4, 1000, 64), (2, 31, 250), (261, 55, 285)])
def test_without_a_workspace(pgk, dtype, shape):
    """The same result whether there is room for segments or not."""
    import torch
    outer, red, inner = shape
    X = torch.randint(-50, 51, shape, device="cuda").to(torch.bfloat16 if dtype == BF16 else torch.float32)
    want = pgk.reduce_max(X, 1)
    v, i = torch.empty_like(want[0]), torch.empty_like(want[1])
    rc = pgk.load_library().pgk_reduce_max(X.data_ptr(), v.data_ptr(), i.data_ptr(), outer, red, inner, dtype, None, 0,
                                           torch.cuda.current_stream().cuda_stream or None)
    torch.cuda.synchronize()
    assert rc == 0 and torch.equal(v, want[0]) and torch.equal(i, want[1])
