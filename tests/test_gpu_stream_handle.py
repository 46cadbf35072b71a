"""The stream handle a call without ``stream`` runs on is that of torch's current stream."""
import threading

import pytest
import torch

from paper_2511_06345_amd import binding

pytestmark = pytest.mark.gpu


def _current():
    return torch.cuda.current_stream().cuda_stream


def test_current_stream_handle():
    side, seen = torch.cuda.Stream(), []
    assert binding._stream_ptr(None) == _current()
    with torch.cuda.stream(side):
        assert binding._stream_ptr(None) == side.cuda_stream != 0
        other = threading.Thread(target=lambda: seen.append((binding._stream_ptr(None), _current())))
        other.start()
        other.join()
    assert seen[0][0] == seen[0][1] != side.cuda_stream
    assert binding._stream_ptr(side) == side.cuda_stream
    x, graph = torch.zeros(8, device="cuda"), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        x.add_(1)
        assert binding._stream_ptr(None) == _current() != 0
