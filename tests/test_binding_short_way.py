"""What the binding does with the answers of its short way (the _call extension), on the CPU with the extension replaced: a call is made
again through the long way only where the short way cannot have enqueued anything."""
import pytest

from paper_2002_01119_amd import psgd

torch = pytest.importorskip("torch")

N, D = 4, 16


def _tensors():
    X, Y, G, Z, H = (torch.zeros(N, D) for _ in range(5))
    nbr, w = psgd.build_mixing(psgd.TOPO_RING, N)
    return X, Y, G, Z, H, torch.from_numpy(nbr), torch.from_numpy(w)


def _calls():
    X, Y, G, Z, H, nbr, w = _tensors()
    return {
        "mix_step": lambda: psgd.mix_step(X, X, G, nbr, w, 0.1),
        "mix_step_d1d": lambda: psgd.mix_step_d1d(X, Y, G, nbr, w, 0.1, Z, H, 0.5),
        "mix_full": lambda: psgd.mix_full(X, X, G, 0.1),
        "build_mixing_device": lambda: psgd.build_mixing_device(psgd.TOPO_RING, N, 0, nbr, w, step_dev=torch.zeros(1, dtype=torch.int64), advance=1),
        "consensus_dist_async": lambda: psgd.consensus_dist_async(X, torch.zeros(1, dtype=torch.float64)),
        "synth_grad": lambda: psgd.synth_grad(X, Z, G, 0.1),
    }


@pytest.fixture
def short_way(monkeypatch):
    """Every function of the extension returns `status[0]` and counts itself."""
    status, made = [psgd.OK], []

    class Extension:
        def __getattr__(self, name):
            return lambda *args: (made.append(name), status[0])[1]

    monkeypatch.setattr(psgd, "_call", Extension())
    return status, made


@pytest.mark.parametrize("name", sorted(_calls()))
def test_a_failure_behind_enqueued_work_is_raised_and_not_tried_again(short_way, monkeypatch, name):
    status, made = short_way
    status[0] = psgd.EHIP
    monkeypatch.setattr(psgd, "_on_current_device", lambda *t: pytest.fail("the long way was taken"))
    with pytest.raises(psgd.PsgdError) as e:
        _calls()[name]()
    assert e.value.code == psgd.EHIP and made == [name]


@pytest.mark.parametrize("rc", [1, psgd.EINVAL, psgd.EALIAS, psgd.EALIGN])
@pytest.mark.parametrize("name", sorted(_calls()))
def test_what_was_not_enqueued_goes_the_long_way(short_way, name, rc):
    status, made = short_way
    status[0] = rc
    with pytest.raises(ValueError):                             # the long way: these are host tensors
        _calls()[name]()
    assert made == [name]


@pytest.mark.parametrize("name", sorted(_calls()))
def test_success_is_the_answer(short_way, name):
    _, made = short_way
    assert _calls()[name]() is None and made == [name]
