"""The scratch a layer keeps for its transposed activations: whose it is.  The library call is replaced by one that notes the
scratch, so this runs without a GPU; tests/test_gpu_linear.py has the same layer on two streams of one."""
import threading
import types

import pytest

torch = pytest.importorskip("torch")

from paper_2310_02065_amd import binding


@pytest.fixture
def layer(monkeypatch):
    """A layer whose calls return the scratch they got; `layer.on` is the current stream, `layer.capturing`
    whether it is being captured."""
    made = object.__new__(binding.Spmm)
    made.handle = types.SimpleNamespace(K=64, R=32, ptr=None)
    made.bias, made.activation = None, "none"
    fresh = getattr(binding, "_KeptScratch", lambda: None)
    made._scratch, made.on, made.capturing = fresh(), 0, False
    monkeypatch.setattr(binding, "_stream_ptr", lambda stream=None: made.on)
    monkeypatch.setattr(binding, "_capturing", lambda stream: made.capturing, raising=False)
    monkeypatch.setattr(binding, "_linear", lambda h, x, bias, act, out, dt, address, nbytes, stream: (address, nbytes))
    return made


X8, X80 = torch.zeros(8, 64), torch.zeros(80, 64)


def test_kept_on_one_stream_and_grown(layer):
    a = layer(X80)
    assert layer(X80) == a and layer(X8) == a and a[1] == 80 * 64 * 2
    big = layer(torch.zeros(88, 64))
    assert big[0] != a[0] and big[1] == 88 * 64 * 2 and layer(X80) == big


def test_streams_have_their_own(layer):
    a = layer(X8)
    layer.on = 1
    b = layer(X8)
    assert a[0] != b[0] and layer(X8) == b
    layer.on = 0
    assert layer(X8) == a


def test_threads_have_their_own(layer):
    a, got = layer(X8), []
    t = threading.Thread(target=lambda: got.append(layer(X8)))
    t.start()
    t.join()
    assert got[0][0] != a[0] and layer(X8) == a


def test_a_captured_call_shares_with_none(layer, monkeypatch):
    made = []
    new = binding._new_scratch
    monkeypatch.setattr(binding, "_new_scratch", lambda *args: made.append(new(*args)) or made[-1])
    a = layer(X8)
    layer.capturing = True
    b, c = layer(X8), layer(X8)
    layer.capturing = False
    assert len({a[0], b[0], c[0]}) == 3 and layer(X8) == a and len(made) == 3


def test_a_bounded_number_is_kept(layer):
    first = layer(X8)
    kept = layer._scratch._buffers[next(iter(layer._scratch._buffers))]
    for layer.on in range(1, 40):
        layer(X8)
    assert len(layer._scratch._buffers) == binding._KeptScratch.LIMIT
    layer.on = 0
    assert layer(X8)[0] != first[0] and kept[1] == first[0]
