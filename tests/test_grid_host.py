"""``Grid.set_state`` on the host: the tensors it reads from live until the
grid's stream has passed the copies, also when a field is refused."""
from types import SimpleNamespace

import pytest

torch = pytest.importorskip("torch")

import paper_2204_01117_amd as U  # noqa: E402
from paper_2204_01117_amd import _lib as L  # noqa: E402


@pytest.mark.parametrize("refused", [None, "u", "w"])
def test_set_state_waits_for_the_copies(monkeypatch, refused):
    events = []
    stream = lambda name: SimpleNamespace(synchronize=lambda: events.append("wait " + name))
    g = U.Grid.__new__(U.Grid)
    g.handle = None
    g.device, g.tstream = "cpu", stream("grid")
    g.torch = SimpleNamespace(cuda=SimpleNamespace(current_stream=lambda device: stream("torch")))
    monkeypatch.setattr(U.Grid, "extent", lambda self, f: (2, 2, 2))
    monkeypatch.setattr(U.Grid, "_dev", lambda self, a, shape: a.reshape(shape))

    def put(handle, field, ptr):
        events.append(L.FIELDS[field])
        return 1 if L.FIELDS[field] == refused else 0

    monkeypatch.setattr(L, "uf_set_field", put)
    state = {f: torch.zeros(8) for f in ("u", "v", "w")}
    if refused is None:
        g.set_state(state)
        assert events == ["wait torch", "u", "v", "w", "wait grid"]
    else:
        with pytest.raises(U.UFError):
            g.set_state(state)
        put_before = ["u", "v", "w"][:["u", "v", "w"].index(refused) + 1]
        assert events == ["wait torch"] + put_before + ["wait grid"]
