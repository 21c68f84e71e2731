"""psgd_mix_step_d1d, the step and the next gradients of the delay-by-one schedule in one pass: bit for bit what psgd_mix_step_deg and
psgd_synth_grad give one after the other, on every route (tiles, ring walk with one and two rows on their way, tables that are not one
ring, other slot counts, an invalid table), and the schedule that uses it against the oracle's delayed trajectory."""
import numpy as np
import pytest

from oracle import psgd_oracle as orc
from paper_2002_01119_amd import inputs as inp

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mods():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2002_01119_amd import d1d, psgd
    psgd.load()
    torch.cuda.set_device(0)
    return psgd, d1d


def _rows(n, d, extra, shift):
    return torch.full((n * (d + extra) + shift,), float("nan"), device="cuda:0").as_strided((n, d), (d + extra, 1), shift)


# n, d, slots (-3: three, not one ring), elements between rows beyond d (0: dense)
@pytest.mark.parametrize("n,d,deg,extra", [
    (1, 3, 3, 0), (2, 1, 3, 2), (8, 40_003, 3, 1), (64, 10_004, 5, 0), (33, 60_001, 13, 3), (16, 1_660_001, 3, 5), (9, 3_700_004, 3, 0),
    (100, 500_003, 3, 0), (101, 400_001, 3, 1), (300, 240_001, 3, 0), (512, 236_000, 3, 4), (64, 420_003, -3, 0), (33, 600_000, -3, 1),
    (16, 1_700_001, 5, 0)])
def test_one_pass_is_the_two_calls(mods, n, d, deg, extra):
    psgd, _ = mods
    if deg == 3:
        nbr, w = psgd.build_mixing(psgd.TOPO_RAND_RING, n, 5, d)
    else:
        rng = np.random.default_rng(n)
        c = rng.random(abs(deg)).astype(np.float32) + np.float32(0.05)
        nbr = np.stack([rng.permutation(n) for _ in range(abs(deg))], axis=1).astype(np.int32)
        w = np.tile((c / c.sum()).astype(np.float32), (n, 1))
    nd, wd = torch.from_numpy(nbr).to("cuda:0"), torch.from_numpy(w).to("cuda:0")
    X, G, Z = (_rows(n, d, extra, extra and k) for k in (1, 2, 3))
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    for t in (X, G, Z):
        t.copy_(torch.empty((n, d), device="cuda:0").normal_(generator=gen))
    Y, H = _rows(n, d, extra, extra), _rows(n, d, 0, 0)
    cd = torch.full((2,), float("nan"), dtype=torch.float64, device="cuda:0")
    psgd.mix_step(X, Y, G, nd, wd, 0.2, delay_mode=1, cdist_out=cd[:1])
    psgd.synth_grad(X, Z, H, 0.3)
    Y1, H1 = _rows(n, d, 2 * extra, extra), _rows(n, d, extra, 0)
    psgd.mix_step_d1d(X, Y1, G, nd, wd, 0.2, Z, H1, 0.3, cdist_out=cd[1:])
    Y2, H2 = _rows(n, d, 0, 0), _rows(n, d, 0, 0)
    psgd.mix_step_d1d(X, Y2, G, nd, wd, 0.2, Z, H2, 0.3)
    torch.cuda.synchronize()
    assert torch.equal(Y1, Y) and torch.equal(Y2, Y) and torch.equal(H1, H) and torch.equal(H2, H)
    assert abs(cd[0].item() - cd[1].item()) <= 1e-12 * cd[0].item()
    assert psgd.device_status() == 0
    # an invalid table: no step, but the next gradients
    nd[n - 1, -1] = n
    Y1.fill_(7.0)
    H1.fill_(7.0)
    psgd.mix_step_d1d(X, Y1, G, nd, wd, 0.2, Z, H1, 0.3, cdist_out=cd[1:])
    torch.cuda.synchronize()
    assert bool((Y1 == 7.0).all()) and torch.equal(H1, H) and torch.isnan(cd[1]) and psgd.device_status() == 1


@pytest.mark.parametrize("n,d", [(8, 40_004), (100, 420_001)])
def test_schedule_in_one_pass_matches_oracle(mods, n, d):
    psgd, d1d = mods
    steps, lr, c = 6, 0.1, 0.3
    X0 = inp.host_normal_f32((n, d), 1.0, 3)
    Z = inp.host_normal_f32((n, d), 0.05, 4)
    tabs = [orc.neighbour_table(orc.TOPO_RAND_RING, n, 9, k) for k in range(steps)]
    want = [X0.astype(np.float64)]
    prev = X0
    for k in range(steps):                                       # the oracle's sparse step, fp64, from its own iterates
        g = c * prev.astype(np.float64) + Z
        x = want[-1]
        y = sum(tabs[k][1][:, s:s + 1].astype(np.float64) * x[tabs[k][0][:, s]] for s in range(3)) - np.float64(np.float32(lr)) * g
        prev = x
        want.append(y)
    tabs_dev = [(torch.from_numpy(a).to("cuda:0"), torch.from_numpy(b).to("cuda:0")) for a, b in tabs]
    X = torch.from_numpy(X0).to("cuda:0")
    noise = torch.from_numpy(Z).to("cuda:0")
    Y, P = torch.full_like(X, float("nan")), torch.full_like(X, float("nan"))
    Gs = [torch.full_like(X, float("nan")) for _ in range(2)]
    cd = torch.zeros(steps, dtype=torch.float64, device="cuda:0")
    torch.cuda.synchronize()
    ms = torch.cuda.Stream()
    run = d1d.DelayByOne(X, Y, P, Gs, noise, lambda k: tabs_dev[k], lr, c, mix_stream=ms)
    assert run.producer_stream is ms
    seen = []
    for k in range(steps):
        out = run.step(cdist_out=cd[k:k + 1], before_mix=seen.append, after_mix=seen.append, more=k + 1 < steps)
    run.finish()
    torch.cuda.synchronize()
    assert seen == [ms] * (2 * steps) and psgd.device_status() == 0
    got = out.cpu().numpy().astype(np.float64)
    scale = max(np.abs(v).max() for v in want)
    assert np.abs(got - want[-1]).max() <= 1e-6 * scale
    ref = orc.consensus_dist(out.cpu().numpy())
    assert abs(cd[-1].item() - ref) <= 1e-6 * ref


def test_one_pass_refuses_arrays_that_overlap(mods):
    psgd, _ = mods
    n, d = 8, 1000
    a = [torch.zeros((n, d), device="cuda:0") for _ in range(5)]
    nbr, w = psgd.build_mixing(psgd.TOPO_RING, n)
    nd, wd = torch.from_numpy(nbr).to("cuda:0"), torch.from_numpy(w).to("cuda:0")
    for X, Y, G, Z, H in ((0, 0, 1, 2, 3), (0, 1, 1, 2, 3), (0, 1, 2, 1, 3), (0, 1, 2, 3, 0), (0, 1, 2, 3, 1), (0, 1, 2, 3, 2), (0, 1, 2, 3, 3)):
        with pytest.raises(psgd.PsgdError) as e:
            psgd.mix_step_d1d(a[X], a[Y], a[G], nd, wd, 0.1, a[Z], a[H], 0.1)
        assert e.value.code == psgd.EALIAS
    with pytest.raises(ValueError):
        psgd.mix_step_d1d(a[0], a[1], a[2].half(), nd, wd, 0.1, a[3], a[4], 0.1)
