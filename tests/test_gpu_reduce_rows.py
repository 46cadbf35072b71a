"""Max reductions along rows (pgk_reduce_max.hip): every number of lanes and chunks that holds a row in registers, the sweep
of longer ones, at the edges between them and at the ends of rows.  Values (bit for bit) and positions are exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pgk():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2511_06345_amd import binding
    binding.load_library()
    return binding


def rows(rng, outer, red, kind):
    if kind == "ties":                                       # the first of many equal ones; zeros of both signs as maxima
        x = rng.integers(-3, 2, (outer, red)).astype(np.float32)
        x[1::2] = np.minimum(x[1::2], 0.0)
        return np.where(x == 0.0, np.where(rng.random(x.shape) < 0.5, np.float32(0.0), np.float32(-0.0)), x)
    if kind == "nan":                                        # none, one or several in a row
        x = rng.integers(-100, 100, (outer, red)).astype(np.float32)
        x[rng.random(x.shape) < 1.0 / red] = np.nan
        x[::7, -1] = np.nan
        return x
    x = np.full((outer, red), -np.inf, np.float32)           # nothing but the type's lowest in most rows
    x[2::3, :] = np.where(rng.random((len(x[2::3]), red)) < 1.0 / red, np.float32(-1e30), x[2::3])
    x[::5, -1] = 3.0
    x[1::5, 0] = np.inf
    return x


# chunks of a row: on each side of the number of lanes, of chunks per lane, of waves and workgroups, of registers and sweeps
CHUNKS = [1, 2, 3, 4, 5, 8, 9, 16, 17, 32, 33, 64, 65, 128, 129, 255, 256, 257, 320, 321, 512, 513, 1024, 1025, 1793, 2048, 2049, 2561, 3072, 3073, 4096, 4097, 6400, 7681, 8192, 8193, 9000]


@pytest.mark.parametrize("chunks", CHUNKS)
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_rows(pgk, dtype, chunks):
    import torch
    vec = 8 if dtype == "bf16" else 4
    for off, less in ((0, 0), (0, 1), (1, 0), (vec - 1, vec - 1)):
        red = chunks * vec - less
        # (a row or some, rows for several workgroups and no whole number of them; many long ones have a way of their own)
        for outer in (3, 301, 1030) if chunks > 2048 else (1, 67):
            kind = ("ties", "nan", "lowest")[(chunks + off + outer) % 3]
            h = rows(np.random.default_rng(chunks * 16 + off), min(outer, 64), red, kind)
            base = torch.empty(outer * red + off, device="cuda", dtype=torch.bfloat16 if dtype == "bf16" else torch.float32)
            x = base[off:].view(outer, red)
            for o in range(0, outer, 64):
                x[o:o + 64] = torch.from_numpy(h[:min(64, outer - o)]).to(x.dtype)
            h = x[:64].float().cpu().numpy()
            nan = np.isnan(h)
            want = np.where(nan.any(1), nan.argmax(1), np.where(nan, -np.inf, h).argmax(1)).astype(np.int64)
            want = torch.from_numpy(np.resize(want, outer)).cuda()
            v, i = pgk.reduce_max(x, 1)
            bits = torch.int16 if dtype == "bf16" else torch.int32
            assert torch.equal(i.view(-1).long(), want), (red, off, outer, kind)
            assert torch.equal(v.view(-1).view(bits), x.gather(1, want[:, None]).view(-1).view(bits)), (red, off, outer, kind)
