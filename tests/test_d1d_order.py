"""What the delay-by-one schedule enqueues, on the CPU with the library's calls and the streams replaced: which gradient goes into which
step, and that no step runs on a gradient that was never produced."""
import contextlib

import pytest

torch = pytest.importorskip("torch")

from paper_2002_01119_amd import d1d


class _Stream:
    def wait_event(self, event):
        pass


class _Event:
    def record(self, stream):
        pass


@pytest.fixture
def calls(monkeypatch):
    """The calls in order: ("G", gradient buffer) for a producer, ("mix", gradient buffer) for a step."""
    made = []
    monkeypatch.setattr(torch.cuda, "stream", lambda s: contextlib.nullcontext())
    monkeypatch.setattr(torch.cuda, "Event", _Event)
    monkeypatch.setattr(torch.cuda, "Stream", lambda **kw: _Stream())
    monkeypatch.setattr(d1d.psgd, "synth_grad", lambda X, Z, G, c, stream: made.append(("G", G)))
    monkeypatch.setattr(d1d.psgd, "mix_step", lambda X, Y, G, nbr, w, lr, **kw: made.append(("mix", G)))
    monkeypatch.setattr(d1d.psgd, "mix_full", lambda X, Y, G, lr, **kw: made.append(("mix", G)))
    monkeypatch.setattr(d1d.psgd, "mix_step_d1d", lambda X, Y, G, nbr, w, lr, Z, H, c, **kw: made.extend([("mix", G), ("G", H)]))
    return made


def _run(form):
    X, Y, P, G0, G1, Z = (torch.zeros(2, 3) for _ in range(6))
    table = None if form == "global averaging" else lambda k: (None, None)
    kw = {"producer_stream": _Stream()} if form == "two streams" else {"overlap": False} if form == "serial" else {}
    return d1d.DelayByOne(X, Y, P, [G0, G1], Z, table, 0.1, 0.3, mix_stream=_Stream(), **kw)


@pytest.mark.parametrize("form", ["one pass", "two streams", "global averaging"])
def test_a_step_without_its_gradient_is_refused(calls, form):
    run = _run(form)
    run.step()
    run.step(more=False)
    before, state = len(calls), (run.k, run.X, run.Y, run.X_prev)
    for _ in range(2):
        with pytest.raises(KeyError):
            run.step()
    assert len(calls) == before and run.k == state[0] and all(a is b for a, b in zip((run.X, run.Y, run.X_prev), state[1:]))


@pytest.mark.parametrize("form", ["one pass", "two streams", "global averaging", "serial"])
def test_every_step_takes_the_gradient_made_for_it(calls, form):
    run = _run(form)
    assert run._one_pass == (form == "one pass")
    steps, produced, used = 5, [], []
    for k in range(steps):
        run.step(more=k + 1 < steps)
    for what, G in calls:
        (produced if what == "G" else used).append(id(G))
    want = [id(run.Gs[k % 2]) for k in range(steps)]
    assert used == want and produced == want
