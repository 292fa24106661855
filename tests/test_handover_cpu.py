"""The order in which the Python front end hands memory of torch's current stream
over to a context's stream, against a library and streams that record their calls
(no device work)."""
import ctypes as ct

import pytest
import torch

from paper_2108_09488_amd import context as M
from paper_2108_09488_amd import inputs as I


class Stream:
    cuda_stream = 0

    def __init__(self, log, name):
        self.log, self.name = log, name

    def wait_stream(self, other):
        self.log.append(("wait", self.name, other.name))


class Library:
    """Every entry point succeeds; sizes are written where they are asked for."""

    def __init__(self, log):
        self.log = log

    def __getattr__(self, name):
        def call(*args):
            if "workspace_bytes" in name:
                args[-1]._obj.value = 256 if name.endswith("_min") else 512
            self.log.append((name, [a.value for a in args if isinstance(a, ct.c_void_p)]))
            return 0
        return call


@pytest.fixture
def fake(monkeypatch):
    log = []
    cur, own = Stream(log, "current"), Stream(log, "own")
    monkeypatch.setattr(M, "lib", lambda lib=Library(log): lib)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: cur)
    monkeypatch.setattr(torch.Tensor, "record_stream", lambda t, s: log.append(("record", s.name, t.data_ptr())))
    return log, cur, own


def _handed_over(log, entry):
    """Whether the own stream waited for the current one before the entry point,
    and the pointers of the call that were recorded on the own stream before it."""
    k = next(k for k, e in enumerate(log) if e[0] == entry)
    before = log[:k]
    recorded = {e[2] for e in before if e[0] == "record" and e[1] == "own"}
    return ("wait", "own", "current") in before, recorded


def _context(own):
    spec = I.config("cfg1")
    return spec, M.Context([M.params_from_spec(spec)], [spec.n], device="cpu", stream=own)


def test_workspace_of_a_context(fake):
    """A context's workspace may be a block that work on the current stream still
    uses, and ade_create writes to it at once."""
    log, _, own = fake
    _, c = _context(own)
    waited, recorded = _handed_over(log, "ade_create")
    assert waited and c.ws.data_ptr() in recorded


def test_inputs_of_the_adjoint(fake):
    """Sensors, observations and the workspace of the adjoint."""
    log, _, own = fake
    spec, c = _context(own)
    xs = torch.zeros((2, 5), dtype=torch.float64)
    obs = torch.zeros(5, dtype=torch.float64)
    del log[:]
    c.adjoint(3, 2, xs, obs)
    waited, recorded = _handed_over(log, "ade_adjoint")
    ptrs = [p for p in next(e[1] for e in log if e[0] == "ade_adjoint") if p]
    assert waited and set(ptrs) <= recorded and len(ptrs) >= 3


def test_nothing_to_hand_over_on_one_stream(fake):
    log, cur, _ = fake
    _context(cur)
    assert not any(e[0] in ("wait", "record") for e in log)


def test_no_memory_for_lists(fake, monkeypatch):
    """A context whose full workspace does not fit takes the least one; where that does
    not fit either, or was asked for, the error is the allocator's."""
    log, _, own = fake
    empty = torch.empty
    limit = [300]

    def scarce(n, **kw):
        if n > limit[0]:
            raise torch.cuda.OutOfMemoryError("out of memory")
        return empty(n, **kw)

    monkeypatch.setattr(torch, "empty", scarce)
    _, c = _context(own)
    assert c.ws_bytes == 256 and c.ws.numel() == 256
    limit[0] = 100
    with pytest.raises(torch.cuda.OutOfMemoryError):
        _context(own)
    limit[0] = 1000
    _, c = _context(own)
    assert c.ws_bytes == 512
