"""The memory the Python forward call takes for a call of few planes: when it may, and from which stream's memory.  Host code only: the
library and torch's device calls are stand-ins, so that cases which would be unsafe on a device are told by what the library is handed."""
import contextlib
import ctypes
import types

import numpy as np
import pytest


class Recorder:
    """Stands in for the library and for torch.cuda; `got` is what the last call handed to the library: workspace, bytes, stream."""
    CURRENT_STREAM, WANTED, ADDRESS = 5, 4096, 0x7000

    def __init__(self, monkeypatch, device=0, current_device=0, capturing=False, pool=(0, 0)):
        import torch
        from paper_2512_07884_amd import binding
        self.binding, self.streams, self.allocated = binding, [], []
        self.x = types.SimpleNamespace(device=f"cuda:{device}", get_device=lambda: device, dtype=torch.bfloat16)
        dims = (1, 8, 50, 70, 2)
        lib = types.SimpleNamespace(gspn_fwd_workspace_bytes=lambda *a: self.WANTED, gspn_scan_fwd_workspace=self.launch)
        monkeypatch.setattr(binding, "load_library", lambda: lib)
        monkeypatch.setattr(binding, "_fwd_args", lambda x, w, lam, u, y, h, G, flags: ([16] * 5 + [None], dims))
        monkeypatch.setattr(binding, "_TORCH", [torch, lambda: current_device, lambda: self.CURRENT_STREAM, lambda: capturing])
        monkeypatch.setattr(binding, "_WORKSPACE_BYTES", {})
        monkeypatch.setattr(torch, "empty", self.empty)
        monkeypatch.setattr(torch.cuda, "memory_snapshot", lambda: [{"address": self.ADDRESS, "total_size": 8192, "segment_pool_id": pool}])
        monkeypatch.setattr(torch.cuda, "stream", self.on_stream)
        monkeypatch.setattr(torch.cuda, "ExternalStream", lambda handle, device: types.SimpleNamespace(cuda_stream=handle, device=device))
        monkeypatch.setattr(torch.cuda, "default_stream", lambda device: types.SimpleNamespace(cuda_stream=0, device=device))

    def empty(self, n, dtype=None, device=None):
        self.allocated.append((n, device, self.streams[-1] if self.streams else None))
        return types.SimpleNamespace(data_ptr=lambda: self.ADDRESS)

    @contextlib.contextmanager
    def on_stream(self, s):
        s.device                                          # (torch's own does not take a stream without one)
        self.streams.append(s.cuda_stream)
        yield
        self.streams.pop()

    def launch(self, *a):
        self.got = a[6], a[7], a[-1]
        return 0

    def scan(self, **k):
        self.got = None
        self.binding.gspn_scan_fwd(self.x, None, None, None, None, **k)
        return self.got


def test_memory_of_the_call(monkeypatch):
    r = Recorder(monkeypatch)
    assert r.scan() == (r.ADDRESS, r.WANTED, r.CURRENT_STREAM)
    assert r.scan(stream=9) == (r.ADDRESS, r.WANTED, 9) and r.allocated[-1] == (r.WANTED, "cuda:0", 9)


@pytest.mark.parametrize("stream", [None, 9])
@pytest.mark.parametrize("pool,taken", [((0, 0), False), ((0, 3), True), ((2, 0), True)])
def test_captured_call_takes_memory_from_the_graphs_own_pool_or_none(pool, taken, stream, monkeypatch):
    """A capture that torch did not begin: its replays would write into what the allocator has handed to others by then."""
    r = Recorder(monkeypatch, capturing=True, pool=pool)
    want = (r.ADDRESS, r.WANTED) if taken else (None, 0)
    assert r.scan(stream=stream)[:2] == want


@pytest.mark.parametrize("device,stream,taken", [
    (0, None, True), (1, None, False), (0, 0, True), (1, 0, False), (1, 9, True),
    (0, types.SimpleNamespace(cuda_stream=9, device="cuda:0", device_index=0), True),
    (1, types.SimpleNamespace(cuda_stream=9, device="cuda:0", device_index=0), False)], ids=str)
def test_memory_is_given_back_in_the_order_of_the_stream_the_call_runs_on(device, stream, taken, monkeypatch):
    """Tensors of device `device` while device 0 is current, on no stream of theirs: the allocator would hand the block on, in the order of
    a stream the call does not run on, while the kernel still writes it."""
    r = Recorder(monkeypatch, device=device, current_device=0)
    assert r.scan(stream=stream)[:2] == ((r.ADDRESS, r.WANTED) if taken else (None, 0))
    assert bool(r.allocated) == taken


@pytest.mark.parametrize("stream", [types.SimpleNamespace(cuda_stream=9), types.SimpleNamespace(cuda_stream=0)], ids=str)
def test_any_object_with_a_stream_handle_names_a_stream(stream, monkeypatch):
    r = Recorder(monkeypatch)
    assert r.scan(stream=stream) == (r.ADDRESS, r.WANTED, stream.cuda_stream)
    assert r.allocated == [(r.WANTED, "cuda:0", stream.cuda_stream)]


@pytest.mark.parametrize("handle", [1, 2])
def test_the_runtimes_stream_names_take_no_memory(handle, monkeypatch):
    """One names another stream in each thread: a block given back by one thread could go to the next while the first still writes it."""
    r = Recorder(monkeypatch)
    assert r.scan(stream=handle) == (None, 0, handle)


@pytest.mark.parametrize("mask", [ctypes.c_uint(15), np.array(15), np.int64(15)], ids=["c_uint", "array", "int64"])
def test_integers_of_other_types_are_asked_about_by_their_value(mask, monkeypatch):
    """What ctypes takes for an unsigned int may have no hash (an array), or be another number the next time (a c_uint)."""
    r = Recorder(monkeypatch)
    asked = []
    ask = lambda *a: asked.append(getattr(a[7], "value", a[7])) or r.WANTED
    monkeypatch.setattr(r.binding.load_library(), "gspn_fwd_workspace_bytes", ask)
    r.scan(dir_mask=mask)
    if isinstance(mask, ctypes.c_uint):
        mask.value = 3
    r.scan(dir_mask=mask)
    assert asked == [15, 3 if isinstance(mask, ctypes.c_uint) else 15]
