"""Where the binding's scratch memory for extends comes from, with torch's streams and allocator replaced by a model of them
(torch.cuda.ExternalStream(0) is a stream of torch's pool, as there)."""
import contextlib
import threading
import types

import pytest
import torch

from paper_2512_23966_amd import binding as B

POOL = 999


class Streams:
    def __init__(self, current):
        self.current, self.owner = current, None

    def install(self, m):
        class Stream:
            def __init__(self, handle):
                self.cuda_stream = handle

        @contextlib.contextmanager
        def use(stream):
            before, self.current = self.current, stream.cuda_stream
            yield
            self.current = before

        def empty(n, **_):
            self.owner = self.current
            return types.SimpleNamespace(numel=lambda: n)
        for name, value in (("Stream", Stream), ("ExternalStream", lambda h: Stream(h or POOL)), ("default_stream", lambda: Stream(0)),
                            ("stream", use), ("is_current_stream_capturing", lambda: False)):
            m.setattr(torch.cuda, name, value)
        m.setattr(torch._C, "_cuda_getDevice", lambda: 0, raising=False)
        m.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: self.current, raising=False)
        m.setattr(torch, "empty", empty)
        return Stream


@pytest.mark.parametrize("current", [0, 640])
@pytest.mark.parametrize("handle", [None, 0, 1, 640, 1280])
@pytest.mark.parametrize("kind", ["handle", "torch", "foreign"])
def test_scratch_memory_is_of_the_stream_of_the_launches(monkeypatch, current, handle, kind):
    streams = Streams(current)
    Stream = streams.install(monkeypatch)
    if handle is None:
        stream = None
    else:
        stream = {"handle": lambda: handle, "torch": lambda: Stream(handle), "foreign": lambda: types.SimpleNamespace(cuda_stream=handle)}[kind]()
    assert B._scratch(64, stream) is not None
    launches = current if handle is None else handle
    # (1 is another handle of the default stream)
    assert streams.owner == (0 if launches == 1 and kind != "torch" else launches) and streams.current == current


def test_the_per_thread_stream_gets_none(monkeypatch):
    streams = Streams(640)
    streams.install(monkeypatch)
    assert B._scratch(64, 2) is None and streams.owner is None


def test_no_memory_is_no_error_and_the_capture_mode_is_as_before(monkeypatch):
    """The allocation happens in HIP's relaxed capture mode of this thread, which is then what it was."""
    Streams(0).install(monkeypatch)
    modes, thread_mode = [], [0]

    def exchange(ref):
        thread_mode[0], ref._obj.value = ref._obj.value, thread_mode[0]

    def empty(n, **_):
        modes.append(thread_mode[0])
        raise torch.OutOfMemoryError("none left")
    monkeypatch.setattr(torch, "empty", empty)
    monkeypatch.setattr(B, "lib", lambda: types.SimpleNamespace(hipThreadExchangeStreamCaptureMode=exchange))
    assert B._scratch(64, None) is None and modes == [2] and thread_mode == [0]


@pytest.mark.parametrize("pattern", [(128, 8192), (1, 7, 128)])
def test_a_refused_call_names_the_entry_point_that_was_called(monkeypatch, pattern):
    monkeypatch.setattr(B, "_scratch", lambda n, stream: types.SimpleNamespace(numel=lambda: n))
    monkeypatch.setattr(B, "_dev_ptr", lambda t, dtype, name: 4096)
    with pytest.raises(B.LozaError, match="^loza_ssa_extend_of_this_name: LOZA_ERR_SHAPE"):
        B._extend_call("loza_ssa_extend_of_this_name", (4096,) * 6, None, (1, 64, 1), None, 65536, 2, 576, 512, pattern, 0.0, None, 640)


SIZES = dict(B=2, Hq=64, S_max=3000, q_len=5, lens=[3000, 1234], pattern=(128, 2000), scale=192 ** -0.5)


def _call(device):
    """A split extend of the sizes above: () -> fresh (out, lse), and call(out, lse, **kw)."""
    from tests.test_gpu_parity_extend import _rand
    s = types.SimpleNamespace(**SIZES)
    assert B.loza_ssa_extend_workspace_bytes(s.B, s.Hq, 1, s.S_max, s.q_len, 576, 512, *s.pattern) > 0
    q, kc = _rand((s.B, s.q_len, s.Hq, 576), 81, torch.bfloat16, device), _rand((s.B, s.S_max, 1, 576), 82, torch.bfloat16, device)
    seqlens = torch.tensor(s.lens, dtype=torch.int32, device=device)
    fresh = lambda: (torch.full((s.B, s.q_len, s.Hq, 512), float("nan"), dtype=torch.bfloat16, device=device),
                     torch.full((s.B, s.Hq, s.q_len), float("nan"), device=device))
    return fresh, lambda out, lse, **kw: B.loza_ssa_extend(q, kc, kc, seqlens, out, lse, *s.pattern, s.scale, **kw)


def _same(a, b):
    return all(torch.equal(x.view(torch.int16), y.view(torch.int16)) for x, y in zip(a, b))


@pytest.mark.gpu
def test_default_stream_by_its_handle_beside_another_current_stream(gpu_device):
    fresh, call = _call(gpu_device)
    ref, got = fresh(), fresh()
    call(*ref)
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.Stream()):
        call(*got, stream=0)
    torch.cuda.synchronize()
    assert _same(got, ref)


@pytest.mark.gpu
def test_a_call_leaves_another_threads_capture_alone(gpu_device):
    fresh, call = _call(gpu_device)
    ref, got, x, side = fresh(), fresh(), torch.zeros(1000, device=gpu_device), torch.cuda.Stream()
    call(*ref)
    x.add_(0)
    errors = []

    def other():
        try:
            with torch.cuda.stream(side):
                call(*got)
        except Exception as e:   # (reported by the thread that waits)
            errors.append(e)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):        # (empties the allocator's cache: the call's scratch memory comes from the driver)
        x.add_(1)
        t = threading.Thread(target=other)
        t.start()
        t.join()
        x.add_(1)
    assert not errors
    for n in (1, 2, 3):
        graph.replay()
        torch.cuda.synchronize()
        assert (x == 2 * n).all()
    assert _same(got, ref)
