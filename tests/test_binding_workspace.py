"""Which calls of mx_gemm_qa the binding gives scratch memory from torch's allocator (no GPU: torch's stream is a stand-in)."""
import types

import pytest
import torch

from paper_2310_10537_amd import binding


@pytest.fixture
def scratch(monkeypatch):
    """The scratch tensor's size for a problem, None where the library allocates by itself."""
    cpu = torch.device("cpu")
    current = types.SimpleNamespace(device=cpu, cuda_stream=11)
    capturing = [False]
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: current)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: capturing[0])

    def size(M, N, K, fa=0, fb=0, stream=None, captured=False):
        capturing[0] = captured
        t = binding._qa_workspace(M, N, K, fa, fb, cpu, stream)
        return None if t is None else t.numel()
    return size


def test_eager_calls_on_the_current_stream_only(scratch):
    assert scratch(1000, 512, 256) == binding.mx_workspace_bytes("gemm_qa", 1000, 512, 256, 0, 0)
    assert scratch(16, 512, 256) is None
    assert scratch(1000, 512, 256, stream=types.SimpleNamespace(cuda_stream=12)) is None
    assert scratch(1000, 512, 256, stream=types.SimpleNamespace(cuda_stream=11)) is not None


def test_none_while_the_stream_is_captured(scratch):
    assert scratch(1000, 512, 256, captured=True) is None


def test_none_where_the_bound_is_far_above_the_need(scratch):
    assert scratch(17, 28672, 8192, 5, 5) is None                       # a 17 x 8192 cast, the product takes none
    assert scratch(65536, 256, 512) is None and scratch(32768, 512, 512) is None   # cast on load: no scratch
    assert scratch(65536, 255, 512) is not None and scratch(32768, 768, 512) is not None and scratch(32767, 512, 512) is not None
