"""The binding's short way (the _call extension) against its long one: same results for what it answers, and what it does not answer
(other types, shapes, devices, subclasses, numbers that are not plain) ends as it does without it."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def psgd():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2002_01119_amd import psgd as m
    m.load()
    torch.cuda.set_device(0)
    assert m._call is not None
    return m


def _both(psgd, monkeypatch, f):
    """f() through the short way and the long one: ("ok", value) or (exception type, text)."""
    got = []
    for short in (True, False):
        with monkeypatch.context() as m:
            if not short:
                m.setattr(psgd, "_call", None)
            try:
                v = f()
                torch.cuda.synchronize()
                got.append(("ok", v))
            except Exception as e:
                got.append((type(e), str(e)))
    return got


@pytest.mark.parametrize("n,d,deg,g,wide", [(8, 1000, 3, torch.float32, 0), (1, 7, 3, torch.bfloat16, 0), (5, 333, 5, torch.bfloat16, 40), (3, 1, 3, torch.float32, 2)])
def test_results_are_the_same(psgd, monkeypatch, n, d, deg, g, wide):
    gen = torch.Generator(device="cuda:0").manual_seed(1)
    pool = torch.empty((4, n, d + wide), device="cuda:0").normal_(generator=gen)
    X, G32, Z = (pool[i, :, wide // 2:wide // 2 + d] for i in range(3))
    G = G32.to(g)
    rng = np.random.default_rng(n)
    nbr = torch.from_numpy(np.stack([rng.permutation(n) for _ in range(deg)], 1).astype(np.int32)).to("cuda:0")
    w = torch.full((n, deg), 1.0 / deg, device="cuda:0")
    s = torch.cuda.Stream()

    def run():
        out = {}
        for st in (None, s):
            c = [torch.zeros(1, dtype=torch.float64, device="cuda:0") for _ in range(4)]
            Y, F, H, P = (torch.zeros((n, d), device="cuda:0") for _ in range(4))
            t, u = torch.zeros((n, 3), dtype=torch.int32, device="cuda:0"), torch.zeros((n, 3), device="cuda:0")
            k = torch.full((1,), 4, dtype=torch.int64, device="cuda:0")
            torch.cuda.synchronize()
            psgd.mix_step(X, Y, G, nbr, w, 0.25, stream=st, cdist_out=c[0])
            psgd.mix_full(X, F, G, 0.25, stream=st, cdist_out=c[1])
            psgd.consensus_dist_async(X, c[2], stream=st)
            psgd.synth_grad(X, Z, H, 0.5, stream=st)
            psgd.mix_step_d1d(X, P, Z, nbr, w, 0.25, Z, F, 0.5, stream=st, cdist_out=c[3])
            psgd.build_mixing_device(1, n, -5, t, u, step_dev=k, step_offset=3, advance=2, stream=st)
            torch.cuda.synchronize()
            out[st is None] = [v.clone() for v in (Y, F, H, P, t, u, k, *c, torch.tensor(psgd.consensus_dist(H)))]
        return out

    a, b = _both(psgd, monkeypatch, run)
    assert a[0] == b[0] == "ok"
    for key in (True, False):
        for x, y in zip(a[1][key], b[1][key]):
            assert torch.equal(x, y)


def test_the_same_calls_are_refused(psgd, monkeypatch):
    n, d = 4, 100
    X, Y, G = (torch.ones((n, d), device="cuda:0") for _ in range(3))
    nbr, w = (torch.from_numpy(a).to("cuda:0") for a in psgd.build_mixing(psgd.TOPO_RING, n))
    cd = torch.zeros(1, dtype=torch.float64, device="cuda:0")
    calls = [
        lambda: psgd.mix_step(X, Y.double(), G, nbr, w, 0.1), lambda: psgd.mix_step(X, Y, G.half(), nbr, w, 0.1),
        lambda: psgd.mix_step(X.cpu(), Y, G, nbr, w, 0.1), lambda: psgd.mix_step(X, Y[:, :50], G, nbr, w, 0.1),
        lambda: psgd.mix_step(X, X, G, nbr, w, 0.1, delay_mode=1), lambda: psgd.mix_step(X, G, G, nbr, w, 0.1),
        lambda: psgd.mix_step(X, Y, G, nbr.long(), w, 0.1), lambda: psgd.mix_step(X, Y, G, nbr, w[:2], 0.1),
        lambda: psgd.mix_step(X, Y, G, nbr, w, 0.1, delay_mode=7), lambda: psgd.mix_step(X, Y, G, nbr, w, 0.1, cdist_out=cd.float()),
        lambda: psgd.mix_step(X.t(), Y.t(), G.t(), nbr, w, 0.1), lambda: psgd.mix_step(X, Y, G, nbr, w, "x"),
        lambda: psgd.mix_full(X, X[:2], G, 0.1), lambda: psgd.consensus_dist_async(X, None), lambda: psgd.consensus_dist_async(X, X), lambda: psgd.consensus_dist(X.t()), lambda: psgd.consensus_dist(X.half()),
        lambda: psgd.build_mixing_device(2, n, 1, nbr, w), lambda: psgd.build_mixing_device(0, 5, 1, nbr, w),
        lambda: psgd.synth_grad(X, Y, X, 0.1), lambda: psgd.synth_grad(X, Y, G[:2], 0.1), lambda: psgd.mix_step(None, Y, G, nbr, w, 0.1),
    ]
    for k, f in enumerate(calls):
        a, b = _both(psgd, monkeypatch, f)
        assert a[0] != "ok" and a == b, k
    # and what only the long way takes is still taken
    for f in (lambda: psgd.mix_step(X, Y, G, nbr, w, 1), lambda: psgd.mix_step(X, Y, G, nbr, w, np.float32(0.1)),
              lambda: psgd.mix_step(torch.nn.Parameter(X, requires_grad=False), Y, G, nbr, w, 0.1),
              lambda: psgd.synth_grad(X.reshape(2, 2, d), Y.reshape(2, 2, d), G.reshape(2, 2, d), 0.1),
              lambda: psgd.build_mixing_device(1, n, 2 ** 64 - 1, nbr, w), lambda: psgd.mix_step(X, Y, G.view(torch.int32).to(torch.int16), nbr, w, 0.1)):
        a, b = _both(psgd, monkeypatch, f)
        assert a[0] == b[0] == "ok"
