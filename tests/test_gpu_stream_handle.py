"""The stream a call is enqueued on is the current device's current stream: the default one, a side stream, a stream that is being captured, and in a thread of
its own, where the current stream is that thread's."""
import threading

import pytest

pytestmark = pytest.mark.gpu


def test_handle_of_the_current_stream():
    import torch
    from paper_2603_21365_amd import tide_route as tr
    torch.zeros(1, device="cuda")
    now = lambda: torch.cuda.current_stream().cuda_stream
    assert tr._stream() == now()
    side = torch.cuda.Stream()
    seen = []
    with torch.cuda.stream(side):
        assert tr._stream() == now() == side.cuda_stream
        t = threading.Thread(target=lambda: seen.append((tr._stream(), now())))
        t.start()
        t.join()
    assert tr._stream() == now() != side.cuda_stream
    assert seen[0][0] == seen[0][1]
    x, g = torch.zeros(4, device="cuda"), torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        x.add_(1)
        seen.append((tr._stream(), now()))
    assert seen[1][0] == seen[1][1]
