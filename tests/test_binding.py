"""What the Python binding checks before it hands a pointer to the library (no GPU)."""
import pytest
import torch

from paper_2106_12372_amd import nrc as N


class _OnDevice(torch.Tensor):
    """A host tensor that passes for a device tensor."""
    is_cuda = True


class _Calls:
    """In the library's place: records the pointer and count of each upload."""

    def __init__(self):
        self.uploads = []

    def nrc_set_weights_device(self, handle, ptr, n, stream):
        self.uploads.append((ptr, n))
        return N.NRC_OK


@pytest.fixture
def upload(monkeypatch):
    calls = _Calls()
    monkeypatch.setattr(N, "lib", calls)
    cache = N.Cache.__new__(N.Cache)
    cache.handle = None
    return lambda w: (cache.set_weights_device(w.as_subclass(_OnDevice), stream=0), calls.uploads.pop())[1]


@pytest.mark.parametrize("shape", [(323 * 64,), (323, 64), (1, 323 * 64), (17, 19, 64), (323 * 64, 1)])
def test_dense_device_weights_are_uploaded_from_where_they_lie(upload, shape):
    w = torch.rand(shape)
    for v in (w, w.transpose(0, -1), w.reshape(-1)[: 64 * 64], w.unsqueeze(0)):
        assert upload(v) == (v.data_ptr(), v.numel())


@pytest.mark.parametrize("view", [
    lambda: torch.rand(1, 64).expand(323, 64),              # 64 elements behind 20,672
    lambda: torch.rand(64, 1).expand(64, 323).t(),
    lambda: torch.rand(323, 128)[:, :64],                   # gaps between the rows
    lambda: torch.rand(323, 128)[:, ::2],
    lambda: torch.rand(646, 64)[::2],
    lambda: torch.rand(64, 324)[:, :323].t(),
    lambda: torch.rand(20672 * 2)[::2],
    lambda: torch.rand(1).expand(20672),
    lambda: torch.rand(400).as_strided((323, 64), (1, 1)),  # rows that overlap
])
def test_device_weights_with_gaps_or_repeats_are_refused(upload, view):
    w = view()
    assert w.numel() == 323 * 64
    with pytest.raises(ValueError, match="contiguous"):
        upload(w)


@pytest.mark.parametrize("private", [True, False])
def test_the_current_stream_without_torchs_private_call(monkeypatch, private):
    class Stream:
        cuda_stream = 0x1230

    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: Stream)
    if private:
        monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 0x4560 + device, raising=False)
    else:
        monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    assert N._stream(None) == (0x4563 if private else 0x1230)
    assert N._stream(Stream) == 0x1230 and N._stream(7) == 7
