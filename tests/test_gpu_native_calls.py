"""The ordinary calls in native code (csrc/pgk_torch.cpp) against the binding's general way, which a call with its own
outputs takes: same bits, same shapes and types, same errors, on the current stream, from several threads, under capture."""
import threading

import numpy as np
import pytest
import torch

from paper_2511_06345_amd import binding as pgk

pytestmark = pytest.mark.gpu
TYPES = [torch.float32, torch.bfloat16]


@pytest.fixture(autouse=True)
def loaded():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    pgk.load_library()
    assert pgk._native is not None


def rand(*shape, dtype=torch.float32, seed=1):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.empty(shape, device="cuda").uniform_(-1, 1, generator=g).to(dtype)


@pytest.mark.parametrize("dtype", TYPES)
@pytest.mark.parametrize("rowsum", [False, True])
@pytest.mark.parametrize("bt", [False, True])
@pytest.mark.parametrize("batch, M, N, K", [(1, 256, 256, 256), (3, 70, 130, 517), (1, 8, 1024, 512), (2, 64, 48, 8200)])
def test_products(dtype, rowsum, bt, batch, M, N, K):
    A, B, bias = rand(batch, M, K, dtype=dtype), rand(batch, *((N, K) if bt else (K, N)), dtype=dtype, seed=2), rand(N, seed=3)
    for fn in (pgk.gemm_fused, pgk.gemm_splitk):
        for b in (bias, None):
            for a, w in ((A, B), (A[0], B[0]) if batch == 1 else (A, B)):
                C, rs = fn(a, w, b, 2, rowsum=rowsum, b_transposed=bt)
                out = torch.empty((batch, M, N), dtype=dtype, device="cuda")
                C2, rs2 = fn(a, w, b, 2, rowsum=rowsum, b_transposed=bt, out=out)
                assert C.shape == C2.shape and C.dtype == C2.dtype and torch.equal(C, C2) and (rs is None) == (not rowsum)
                assert rs is None or (rs.dtype == torch.float32 and rs.shape == (batch, M) and torch.equal(rs, rs2))


@pytest.mark.parametrize("dtype", TYPES)
def test_reductions_and_convolutions(dtype):
    X = rand(3, 1000, 7, dtype=dtype)
    for dim in (0, 1, 2, -1, 4):
        v, i = pgk.reduce_max(X, dim)
        v2, i2 = pgk.reduce_max(X, dim, out=torch.empty(v.shape, dtype=dtype, device="cuda"))
        assert torch.equal(v, v2) and torch.equal(i, i2) and i.dtype == torch.int32 and v.dtype == dtype
        assert pgk.reduce_max(X, dim, want_idx=False)[1] is None
    x, w, bias = rand(2, 40, 777, dtype=dtype), rand(33, 40, 3, dtype=dtype, seed=2), rand(33, seed=3)
    for stride, pad, dilation in ((1, 0, 1), (2, 1, 2), (1, 1, 1)):
        y = pgk.conv1d(x, w, bias, 1, stride, pad, dilation)
        assert torch.equal(y, pgk.conv1d(x, w, bias, 1, stride, pad, dilation, out=torch.empty_like(y))) and y.dtype == dtype


def test_what_is_refused_is_refused_the_same_way():
    A, B, bias = rand(64, 64), rand(64, 64, seed=2), rand(64, seed=3)
    w = rand(4, 3, 5)
    for error, call in ((TypeError, lambda: pgk.gemm_fused(A, B.bfloat16(), bias, 0)), (ValueError, lambda: pgk.gemm_fused(A.cpu(), B, bias, 0)),
                        (ValueError, lambda: pgk.gemm_fused(A.t(), B, bias, 0)), (ValueError, lambda: pgk.gemm_fused(A, B[:32], bias, 0)),
                        (ValueError, lambda: pgk.gemm_fused(A, B, bias[:8], 0)), (ValueError, lambda: pgk.gemm_fused(A, B, bias.bfloat16(), 0)),
                        (TypeError, lambda: pgk.gemm_fused(A.double(), B.double(), None, 0)), (pgk.PgkError, lambda: pgk.gemm_fused(A, B, bias, 9)),
                        (pgk.PgkError, lambda: pgk.gemm_splitk(A, B, bias, 0, splits=-1)), (ValueError, lambda: pgk.reduce_max(A.t(), 0)),
                        (TypeError, lambda: pgk.reduce_max(A.int(), 0)), (pgk.PgkError, lambda: pgk.reduce_max(A[:0], 1)),
                        (ValueError, lambda: pgk.conv1d(A, w, None)), (ValueError, lambda: pgk.conv1d(rand(1, 3, 4), w, None)),
                        (pgk.PgkError, lambda: pgk.conv1d(rand(1, 3, 40), w, None, 7))):
        with pytest.raises(error):
            call()
    with pytest.raises(pgk.PgkError, match="pgk_gemm_fused_bt"):
        pgk.gemm_fused_bt(A, B, bias, -3)
    # numbers that are no plain ints go the general way, and are taken or refused as there
    C, _ = pgk.gemm_fused(A, B, bias, np.int64(1), rowsum=np.bool_(True))
    assert torch.equal(C, pgk.gemm_fused(A, B, bias, 1)[0])


def test_streams_threads_and_capture():
    A, B, bias = rand(300, 517), rand(517, 400, seed=2), rand(400, seed=3)
    want, want_rs = pgk.gemm_fused(A, B, bias, 3)
    side, out = torch.cuda.Stream(), []
    torch.cuda.synchronize()

    def work():
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(20):
                got = pgk.gemm_fused(A, B, bias, 3)
            torch.cuda.current_stream().synchronize()
            out.append(got)
    threads = [threading.Thread(target=work) for _ in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert len(out) == 4 and all(torch.equal(C, want) and torch.equal(rs, want_rs) for C, rs in out)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            C, rs = pgk.gemm_fused(A, B, bias, 3)
    for k in range(3):
        A.uniform_(-1, 1)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        again = pgk.gemm_fused(A, B, bias, 3)
        assert torch.equal(C, again[0]) and torch.equal(rs, again[1])
