"""scale_ on a tensor of another device than the current one (CPU only, with the GPU side
of torch and the library replaced)."""
import contextlib
import ctypes
import types

import pytest

torch = pytest.importorskip("torch")

from paper_2507_15121_amd import api  # noqa: E402


class _OnGpu:
    """A tensor's place without the tensor."""

    def __init__(self, dtype, index, n=8):
        self.dtype, self.n = dtype, n
        self.is_cuda, self.device = True, torch.device("cuda", index)

    def is_contiguous(self):
        return True

    def numel(self):
        return self.n

    def data_ptr(self):
        return 4096


class _Gpu:
    def __init__(self, current):
        self.current, self.calls = current, []
        self.float32, self.float64 = torch.float32, torch.float64
        self.cuda = types.SimpleNamespace(device=self._device, current_device=lambda: self.current)
        self._C = types.SimpleNamespace(_cuda_getDevice=lambda: self.current,
                                        _cuda_getCurrentRawStream=lambda d: 100 + d)

    @contextlib.contextmanager
    def _device(self, d):
        before, self.current = self.current, torch.device(d).index if not isinstance(d, int) else d
        try:
            yield
        finally:
            self.current = before

    def amped_scale(self, x, n, s, stream):
        self.calls.append((self.current, ctypes.cast(stream, ctypes.c_void_p).value))
        return 0


@pytest.mark.parametrize("current,index", [(0, 0), (0, 1), (2, 0)])
def test_runs_where_the_tensor_is(monkeypatch, current, index):
    gpu = _Gpu(current)
    monkeypatch.setattr(api, "_torch", lambda: gpu)
    monkeypatch.setattr(api, "lib", lambda: gpu)
    x = _OnGpu(torch.float32, index)
    assert api.scale_(x, _OnGpu(torch.float64, index, 1)) is x
    assert gpu.calls == [(index, 100 + index)]
    assert gpu.current == current


def test_factor_on_another_device(monkeypatch):
    gpu = _Gpu(0)
    monkeypatch.setattr(api, "_torch", lambda: gpu)
    monkeypatch.setattr(api, "lib", lambda: gpu)
    with pytest.raises(ValueError):
        api.scale_(_OnGpu(torch.float32, 0), _OnGpu(torch.float64, 1, 1))
    assert not gpu.calls
