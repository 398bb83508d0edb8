"""The native host side of a call (csrc/host/llla_host.cpp) against the Python one: the same bits for every form that it takes, and the same
errors for what it leaves to the other."""
import itertools
import sys
import threading
import time

import pytest
import torch

import paper_2510_01450_amd as llla
from paper_2510_01450_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda"


class _Absent:
    def forward(self, *args):
        return NotImplemented

    decode = forward


class _Recorder:
    """The native side, and what became of the calls that it was offered: its own result, a status of the C ABI, or left to Python."""

    def __init__(self, host):
        self.host, self.seen = host, []

    def _note(self, r):
        self.seen.append("left" if r is NotImplemented else "status" if type(r) is int else "served")
        return r

    def forward(self, *args):
        return self._note(self.host.forward(*args))

    def decode(self, *args):
        return self._note(self.host.decode(*args))


def _both(monkeypatch, call, native="served"):
    """A call as it is, which the native side has to take as `native` says, and with that side leaving everything to Python; their results or errors."""
    out = []
    recorder = _Recorder(binding._load_host())
    for side in (recorder, _Absent()):
        with monkeypatch.context() as m:
            m.setattr(binding, "_host", side)
            try:
                r = call()
                out.append(tuple(r) if isinstance(r, tuple) else (r,))
            except Exception as e:           # noqa: BLE001
                out.append((type(e), str(e)))
    assert recorder.seen == [native], recorder.seen
    return out


@pytest.mark.parametrize("dtype,d", [(torch.float32, 16), (torch.bfloat16, 64), (torch.float32, 128)])
def test_forward_forms(monkeypatch, dtype, d):
    g = torch.Generator(device=DEV).manual_seed(d)
    B, H, n = 2, 3, 70
    Q, K, V = (torch.randn(B, H, n, 2 * d, generator=g, device=DEV, dtype=dtype)[..., :d] for _ in range(3))
    ridge = torch.full((B, H, n), 1e-2, device=DEV)
    ws = torch.empty(max(256, llla.forward_workspace_bytes(B, H, n, d, dtype)), dtype=torch.uint8, device=DEV)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    for lam, causal, stats, odt, w, st in itertools.product((1e-2, ridge), (True, False), (False, True), (None, torch.bfloat16), (None, ws), (None, side)):
        a, b = _both(monkeypatch, lambda: llla.llla_forward(Q, K, V, lam, d ** -0.5, causal=causal, out_dtype=odt, workspace=w, stream=st, return_stats=stats))
        torch.cuda.synchronize()
        assert len(a) == len(b) == (3 if stats else 1)
        for x, y in zip(a, b):
            assert x.dtype == y.dtype and x.shape == y.shape and torch.equal(x, y)
    out = torch.empty(B, H, n, d, device=DEV, dtype=torch.bfloat16)
    for r in _both(monkeypatch, lambda: llla.llla_forward(Q, K, V, 1e-2, 1.0, out=out)):
        assert r[0] is out


@pytest.mark.parametrize("dtype,d", [(torch.float32, 64), (torch.bfloat16, 32), (torch.bfloat16, 128)])
def test_decode_forms(monkeypatch, dtype, d):
    g = torch.Generator(device=DEV).manual_seed(d)
    B, H, L = 2, 3, 600
    q = torch.randn(B, H, d, generator=g, device=DEV, dtype=dtype)
    K, V = (torch.randn(B, H, L, d, generator=g, device=DEV, dtype=dtype) for _ in range(2))
    lens = torch.tensor([40, L], dtype=torch.int32, device=DEV)
    ws = torch.empty(max(256, llla.decode_workspace_bytes(B, H, L, d, dtype)), dtype=torch.uint8, device=DEV)
    for sl, odt, w, path in itertools.product((None, lens), (None, torch.bfloat16), (None, ws), ("auto", "valu")):
        a, b = _both(monkeypatch, lambda: llla.llla_decode(q, K, V, 1e-2, d ** -0.5, seqlens=sl, out_dtype=odt, workspace=w, path=path))
        assert a[0].dtype == b[0].dtype and torch.equal(a[0], b[0])
    out = torch.empty(B, H, d, device=DEV)
    for r in _both(monkeypatch, lambda: llla.llla_decode(q, K, V, 1e-2, 1.0, out=out)):
        assert r[0] is out


def test_mistakes_are_worded_alike(monkeypatch):
    t = torch.zeros(1, 2, 40, 16, device=DEV)
    q = torch.zeros(1, 2, 16, device=DEV)
    cases = [lambda: llla.llla_forward(t, t, t.double(), 0.1, 1.0), lambda: llla.llla_forward(t, t[:, :, :39], t, 0.1, 1.0),
             lambda: llla.llla_forward(t, t.cpu(), t, 0.1, 1.0), lambda: llla.llla_forward(t[0], t[0], t[0], 0.1, 1.0),
             lambda: llla.llla_forward(t, t, t, 0.1, 1.0, path="other"), lambda: llla.llla_forward(t, t, t, 0.1, 1.0, out_dtype=torch.float16),
             lambda: llla.llla_forward(t, t, t, -1.0, 1.0), lambda: llla.llla_forward(t, t, t, torch.ones(3, device=DEV), 1.0),
             lambda: llla.llla_forward(t.transpose(2, 3), t.transpose(2, 3), t.transpose(2, 3), 0.1, 1.0), lambda: llla.llla_forward(t, t, t, "x", 1.0),
             lambda: llla.llla_forward(t[..., 1:], t[..., 1:], t[..., 1:], 0.1, 1.0), lambda: llla.llla_forward([], t, t, 0.1, 1.0),
             lambda: llla.llla_decode(q, t, t, 0.1, 1.0, seqlens=torch.ones(1, device=DEV)), lambda: llla.llla_decode(q[:, :1], t, t, 0.1, 1.0),
             lambda: llla.llla_decode(q, t, t, 0.0, 1.0), lambda: llla.llla_decode(q, t, t, 0.1, 1.0, out=q.to(torch.float16))]
    refused_by_the_library = (6, 10, 14)                 # ridge, alignment, ridge
    for i, call in enumerate(cases):
        a, b = _both(monkeypatch, call, "status" if i in refused_by_the_library else "left")
        assert isinstance(a[0], type) and a == b, (i, a, b)


def test_integers_and_scalars_serve_as_numbers(monkeypatch):
    import numpy as np
    t = torch.randn(1, 2, 40, 16, device=DEV)
    a, b = _both(monkeypatch, lambda: llla.llla_forward(t, t, t, 1, np.float64(1.0), causal=1), "left")
    want, _ = _both(monkeypatch, lambda: llla.llla_forward(t, t, t, 1.0, 1.0))
    assert torch.equal(want[0], a[0]) and torch.equal(want[0], b[0])


def _try_to_allocate(call, tries):
    """Whether another thread gets to run while `call` fails to allocate; Python itself switches threads only where one gives way."""
    ran, stop = [0], threading.Event()

    def other():
        while not stop.is_set():
            ran[0] += 1
            time.sleep(1e-4)
    thread = threading.Thread(target=other)
    interval = sys.getswitchinterval()
    thread.start()
    try:
        sys.setswitchinterval(1000.)
        before = ran[0]
        for _ in range(tries):
            try:
                call()
            except torch.cuda.OutOfMemoryError:
                pass
            else:
                raise AssertionError("there was room")
            if ran[0] != before:
                return True
        return False
    finally:
        sys.setswitchinterval(interval)
        stop.set()
        thread.join()


def test_allocation_holds_up_no_other_thread():
    """torch's allocator can take its time (it synchronises and frees what it caches before it gives up, as here under a limit): Python's lock
    is not held meanwhile."""
    t = torch.zeros(1, 1, 1 << 20, 16, device=DEV)
    q, cache = torch.zeros(4, 8, 128, device=DEV), torch.zeros(4, 8, 2048, 128, device=DEV)
    assert llla.decode_workspace_bytes(4, 8, 2048, 128, torch.float32) > 32 << 20
    calls = [lambda: llla.llla_forward(t, t, t, 0.1, 1.0), lambda: llla.llla_decode(q, cache, cache, 0.1, 1.0)]
    small = torch.zeros(1, 1, 40, 16, device=DEV)
    llla.llla_forward(small, small, small, 0.1, 1.0)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    torch.cuda.set_per_process_memory_fraction(torch.cuda.memory_reserved() / total)
    try:
        for i, call in enumerate(calls):
            assert _try_to_allocate(call, 200), i
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
