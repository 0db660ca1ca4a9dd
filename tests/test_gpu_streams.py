"""The stream a call runs on: torch's current one at call time (the default
stream, a side stream, the stream under capture) or the handle's own."""
import pytest
import torch

import paper_2301_13062_amd as cp

pytestmark = pytest.mark.gpu


def test_stream_of_a_call(gpu):
    s = cp.CartPoleStates(64)
    side = torch.cuda.Stream()
    assert (s.handle().stream or 0) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert s.handle().stream == side.cuda_stream == torch.cuda.current_stream().cuda_stream
    assert (s.handle().stream or 0) == torch.cuda.default_stream().cuda_stream
    cp.cp_init(s, 0)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        assert s.handle().stream == torch.cuda.current_stream().cuda_stream
        cp.cp_step(s, torch.ones(64, dtype=torch.uint8, device="cuda"))
    s.stream = side
    assert s.handle().stream == side.cuda_stream
