"""Where the binding takes a call's scratch from (CPU: torch's stream and allocation calls are
recorded, nothing runs on a GPU)."""

import contextlib
import types

import pytest

import paper_2606_16317_amd as dsa


@pytest.fixture
def recorded(monkeypatch):
    torch = pytest.importorskip("torch")
    log = []

    @contextlib.contextmanager
    def on(stream):
        log.append(("stream", stream.cuda_stream, str(stream.device)))
        yield

    def empty(n, dtype, device):
        log.append(("empty", n, str(device)))
        return types.SimpleNamespace(data_ptr=lambda: 4096)

    def external(handle, device):
        return types.SimpleNamespace(cuda_stream=handle, device=device)

    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: False)
    monkeypatch.setattr(torch.cuda, "stream", on)
    monkeypatch.setattr(torch.cuda, "ExternalStream", external)
    monkeypatch.setattr(torch, "empty", empty)
    return log


def test_scratch_belongs_to_the_device_of_the_launch(recorded):
    """Tensors on cuda:1: without a stream the kernels go to the current device's current
    stream, with one to that stream's device."""
    dsa._workspace(64, "cuda:1", None)
    assert recorded == [("empty", 64, "cuda")]
    recorded.clear()
    dsa._workspace(64, "cuda:1", types.SimpleNamespace(cuda_stream=7, device="cuda:0"))
    assert recorded == [("stream", 7, "cuda:0"), ("empty", 64, "cuda:0")]
    recorded.clear()
    dsa._workspace(64, "cuda:1", types.SimpleNamespace(cuda_stream=8))
    assert recorded == [("stream", 8, "cuda:1"), ("empty", 64, "cuda:1")]
    assert dsa._workspace(0, "cuda:1", None) is None


@pytest.mark.parametrize("stream", [None, types.SimpleNamespace(cuda_stream=7, device="cuda:0")])
def test_optional_scratch_is_left_out_under_capture_and_without_memory(recorded, monkeypatch,
                                                                       stream):
    torch = pytest.importorskip("torch")
    assert dsa._workspace(64, "cuda:0", stream, optional=True) is not None

    def full(*args, **kw):
        raise torch.cuda.OutOfMemoryError("full")

    with monkeypatch.context() as m:
        m.setattr(torch, "empty", full)
        assert dsa._workspace(64, "cuda:0", stream, optional=True) is None
        with pytest.raises(torch.cuda.OutOfMemoryError):
            dsa._workspace(64, "cuda:0", stream)
    recorded.clear()
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: True)
    assert dsa._workspace(64, "cuda:0", stream, optional=True) is None
    assert not any(entry[0] == "empty" for entry in recorded)
    assert dsa._workspace(64, "cuda:0", stream) is not None     # what the call needs, it gets
