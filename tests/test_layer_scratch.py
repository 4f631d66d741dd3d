"""The scratch a layer keeps for its transposed activations: whose it is.  The library call is replaced by one that notes the
scratch, so this runs without a GPU; tests/test_gpu_linear.py has the same layer on two streams of one."""
import threading
import types

import pytest

torch = pytest.importorskip("torch")

from paper_2310_02065_amd import binding


@pytest.fixture
def layer(monkeypatch):
    """A layer whose calls return (address, bytes) of their scratch; `layer.on` is the current stream, `layer.capturing`
    whether it is being captured."""
    made = object.__new__(binding.Spmm)
    made.handle = types.SimpleNamespace(K=64, R=32, ptr=None)
    made.bias, made.activation = None, "none"
    fresh = getattr(binding, "_KeptScratch", lambda: None)
    made._scratch, made.on, made.capturing = fresh(), 0, False
    monkeypatch.setattr(binding, "_stream_ptr", lambda stream=None: made.on)
    monkeypatch.setattr(binding, "_capturing", lambda stream: made.capturing, raising=False)
    monkeypatch.setattr(binding, "_linear", lambda h, x, bias, act, out, dt, scratch, stream: scratch)
    return made


X8, X80 = torch.zeros(8, 64), torch.zeros(80, 64)


def test_kept_on_one_stream_and_grown(layer):
    a = layer(X80)
    assert layer(X80) is a and layer(X8) is a and a.numel() == 80 * 64 * 2
    big = layer(torch.zeros(88, 64))
    assert big is not a and big.numel() == 88 * 64 * 2 and layer(X80) is big


def test_streams_have_their_own(layer):
    a = layer(X8)
    layer.on = 1
    b = layer(X8)
    assert a.data_ptr() != b.data_ptr() and layer(X8) is b
    layer.on = 0
    assert layer(X8) is a


def test_threads_have_their_own(layer):
    a, got = layer(X8), []
    t = threading.Thread(target=lambda: got.append(layer(X8)))
    t.start()
    t.join()
    assert got[0].data_ptr() != a.data_ptr() and layer(X8) is a


def test_a_captured_call_shares_with_none(layer):
    a = layer(X8)
    layer.capturing = True
    b, c = layer(X8), layer(X8)
    layer.capturing = False
    assert len({a.data_ptr(), b.data_ptr(), c.data_ptr()}) == 3 and layer(X8) is a


def test_a_bounded_number_is_kept(layer):
    first = layer(X8)
    for layer.on in range(1, 40):
        layer(X8)
    assert len(layer._scratch._buffers) == binding._KeptScratch.LIMIT
    layer.on = 0
    assert layer(X8) is not first
