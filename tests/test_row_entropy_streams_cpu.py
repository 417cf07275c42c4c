"""Which stream and which device a row_entropy call uses, without a GPU: the binding runs against a
stand-in for torch that keeps track of current streams, of the stream each allocation belongs to,
and of what a launch was given."""
import sys
from contextlib import contextmanager
from types import SimpleNamespace

import pytest

from paper_2603_18489_amd import binding


class Stream:
    def __init__(self, raw, device):
        self.cuda_stream, self.device, self.waited = raw, device, 0

    def synchronize(self):
        self.waited += 1


class Tensor:
    def __init__(self, torch, shape, dtype, device):
        self.shape, self.dtype, self.device = shape, dtype, device
        self.owner = torch.current[device]      # the caching allocator's rule: the current stream's pool
        self.recorded = []
        torch.tensors.append(self)
        self.ptr = 256 * len(torch.tensors)

    def stride(self, i):
        return self.shape[1] if i == 0 else 1

    def get_device(self):
        return self.device

    def data_ptr(self):
        return self.ptr

    def is_contiguous(self):
        return True

    def record_stream(self, s):
        self.recorded.append(s)


class Torch:
    """current device, one current stream a device, allocations, launches"""
    float32, uint8 = "float32", "uint8"

    def __init__(self):
        self.dev, self.tensors, self.launches = 0, [], []
        self.current = {d: Stream(1000 + d, d) for d in (0, 1)}
        idx = lambda d: self.dev if d is None else d
        self.cuda = SimpleNamespace(
            current_device=lambda: self.dev, stream=self._stream, device=self._device,
            current_stream=lambda d=None: self.current[idx(d)])
        self._C = SimpleNamespace(_cuda_getCurrentRawStream=lambda d: self.current[d].cuda_stream)

    @contextmanager
    def _device(self, d):
        old, self.dev = self.dev, d
        yield
        self.dev = old

    @contextmanager
    def _stream(self, s):
        old, self.current[s.device] = self.current[s.device], s
        with self._device(s.device):
            yield
        self.current[s.device] = old

    def empty(self, shape, dtype, device):
        return Tensor(self, shape if isinstance(shape, tuple) else (shape,), dtype, device)

    # the library's entry points
    def ec_row_entropy_workspace_bytes(self, rows, vocab):
        return 4096

    def ec_row_entropy(self, logits, rows, vocab, ld, stats, ws, ws_bytes, stream):
        by_ptr = {t.ptr: t for t in self.tensors}
        self.launches.append((by_ptr[stats], by_ptr[ws], stream, self.dev))
        return 0

    def ec_row_entropy_noalloc(self, logits, rows, vocab, ld, stats, stream):
        self.launches.append((None, None, stream, self.dev))
        return 0


@pytest.fixture
def torch(monkeypatch):
    t = Torch()
    monkeypatch.setitem(sys.modules, "torch", t)
    monkeypatch.setattr(binding, "_lib", t)
    return t


def test_the_workspace_belongs_to_the_stream_that_uses_it(torch):
    """A call on the current stream returns while its kernels are pending, and its workspace goes back
    to that stream's pool: a call on another stream must not take its own from there."""
    z = Tensor(torch, (64, 40000), "float32", 0)
    here, side = torch.current[0], Stream(7, 0)
    binding.row_entropy(z)
    r = binding.row_entropy(z, stream=side)
    binding.row_entropy(z, stream=here)
    for stats, ws, raw, _ in torch.launches:
        assert ws.owner.cuda_stream == raw and stats.owner.cuda_stream == raw
    assert [l[2] for l in torch.launches] == [1000, 7, 1000]
    assert side.waited == 1 and torch.current[0] is here
    # the caller goes on with the result on its own stream
    assert r is torch.launches[1][0] and r.recorded == [here]


def test_logits_on_a_device_that_is_not_current(torch):
    """The kernels run on the device of the logits, on that device's current stream: the one that result
    and workspace belong to."""
    z = Tensor(torch, (64, 40000), "float32", 1)
    r = binding.row_entropy(z)
    stats, ws, raw, dev = torch.launches.pop()
    assert (raw, dev) == (1001, 1) and r is stats
    assert stats.owner.cuda_stream == ws.owner.cuda_stream == raw
    binding.row_entropy_noalloc(z, r)
    assert torch.launches.pop()[2:] == (1001, 1)
    side = Stream(8, 1)
    r = binding.row_entropy(z, stream=side)
    stats, ws, raw, dev = torch.launches.pop()
    assert (raw, dev) == (8, 1) and stats.owner is ws.owner is side and r.recorded == [torch.current[1]]
    binding.row_entropy_noalloc(z, r, stream=side)
    assert torch.launches.pop()[2:] == (8, 1)
    assert torch.dev == 0



def test_current_stream_without_the_short_lookup(torch):
    """torch's undocumented lookup of the current stream is used only where it exists."""
    del torch._C._cuda_getCurrentRawStream
    binding.row_entropy(Tensor(torch, (2, 100), "float32", 0))
    assert torch.launches.pop()[2] == 1000
