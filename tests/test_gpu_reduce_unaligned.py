"""Max reduction over rows that do not start on 16-byte boundaries: read in 16-byte chunks all the
same, with the elements before and behind them apart.  Exact against the oracle (values and first
positions), for every start of X, at the edges of chunks, sweeps, segments and row groups."""
import numpy as np
import pytest

from paper_2511_06345_amd import inputs as gen

pytestmark = pytest.mark.gpu
F32, BF16 = gen.F32, gen.BF16


@pytest.fixture(scope="module")
def pgk():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2511_06345_amd import binding
    binding.load_library()
    return binding


# outer, red, inner: few lanes per row, a wave per row, a workgroup per row, segments of a row; the strided kernel
ROWS = [(300, 129, 1), (65, 131, 1), (33, 1000, 1), (40, 1031, 1), (9, 2049, 1), (7, 4103, 1), (700, 8199, 1), (3, 70001, 1), (1, 1000003, 1)]
COLS = [(3, 5, 65), (2, 33, 67), (1, 700, 129), (5, 64, 511), (2, 100, 1025)]


def check(pgk, oracle, X, start, dtype):
    import torch
    flat = np.concatenate([X.reshape(-1)[:start], X.reshape(-1)])
    d = torch.from_numpy(flat.view(np.int16) if dtype == BF16 else flat).cuda()
    d = (d.view(torch.bfloat16) if dtype == BF16 else d)[start:].view(*X.shape)
    ref_v, ref_i = oracle.reduce_max(X, 1)
    v, i = pgk.reduce_max(d, 1)
    torch.cuda.synchronize()
    got = v.float().cpu().numpy()                       # (exact: a maximum is one of the values)
    assert np.array_equal(got, np.asarray(ref_v, dtype=np.float32), equal_nan=True), (X.shape, start)
    assert np.array_equal(i.cpu().numpy(), ref_i), (X.shape, start)


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("shape", ROWS + COLS)
def test_unaligned_rows(pgk, oracle, dtype, shape):
    n = shape[0] * shape[1] * shape[2]
    x = gen.uniform(gen.tensor_seed(98, 1, n), n, -1.0, 1.0)
    x = (gen.f32_to_bf16_bits(x) if dtype == BF16 else x).reshape(shape)
    for start in range(8 if dtype == BF16 else 4):
        check(pgk, oracle, x, start, dtype)


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("shape", [(40, 133, 1), (40, 1031, 1), (20, 4103, 1), (2, 70001, 1), (3, 37, 67)])
def test_unaligned_rows_special_values(pgk, oracle, dtype, shape):
    """Maxima and NaNs in the first and last places of rows, rows of nothing but -inf, ties."""
    outer, red, inner = shape
    x = gen.uniform(gen.tensor_seed(98, 2), outer * red * inner, -1.0, 0.5).reshape(shape)
    x[0, 0], x[0, red - 1] = 2.0, 2.0
    x[1, red - 1] = 2.0
    x[-1] = -np.inf
    if outer > 8:
        x[2] = -np.inf
        x[2, red - 1] = -1e30
        x[3, red - 1] = np.nan
        x[4, 1], x[4, red - 2] = np.nan, 3.0
        x[5] = 0.25
        x[6, 1], x[6, 2] = 2.0, 2.0
        x[7] = np.nan
    x = gen.f32_to_bf16_bits(x) if dtype == BF16 else x
    for start in (0, 1, 3):
        check(pgk, oracle, x, start, dtype)


# unaligned rows of a strided reduction that are read in chunks because there is enough to do: segments of the
# reduced range, one pass, a last lane whose chunk overlaps its neighbour's, lanes without a chunk, several tiles
BIG_COLS = {F32: [(3, 5000, 321), (700, 63, 133), (300, 130, 259), (2, 9001, 241)],
            BF16: [(3, 7000, 517), (600, 150, 129), (1100, 75, 131), (40, 250, 1025)]}


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("which", range(4))
def test_unaligned_columns_in_chunks(pgk, oracle, dtype, which):
    shape = BIG_COLS[dtype][which]
    n = shape[0] * shape[1] * shape[2]
    x = gen.uniform(gen.tensor_seed(98, 3, n), n, -1.0, 1.0)
    x = (gen.f32_to_bf16_bits(x) if dtype == BF16 else x).reshape(shape)
    for start in (0, 1):
        check(pgk, oracle, x, start, dtype)
