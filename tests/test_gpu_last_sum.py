"""The distance's last sum, made by the workgroup that is done last: workgroup counts on both sides of where tickets are drawn in two
steps, the same counters launch after launch, graph replays between eager calls, and calls behind some that overlapped by mistake."""
import numpy as np
import pytest
import torch

from paper_2002_01119_amd import psgd

pytestmark = pytest.mark.gpu
LANES, COLS = 256, 4          # of a workgroup of the distance kernel for few learners; columns of a lane
TICKETS = 256                 # draws and launches enough that a counter left off zero would show


def _reference(X):
    x = X.double()
    return float((x - x.mean(0, keepdim=True)).square().sum())


@pytest.mark.parametrize("groups", [1, 2, 16, 17, 63, 64, 65, 66, 79, 80, 81, 512, 513, 1100])
@pytest.mark.parametrize("odd", [0, 3])
def test_workgroup_counts(groups, odd):
    n, d = 3, groups * LANES * COLS - odd
    gen = torch.Generator(device="cuda:0").manual_seed(groups)
    X = torch.randn(n, d, device="cuda:0", generator=gen)
    want = _reference(X)
    out = torch.full((4,), float("nan"), dtype=torch.float64, device="cuda:0")
    for k in range(4):
        psgd.consensus_dist_async(X, out[k:k + 1])
    got = out.tolist()
    # fp64 sums of n d squares in any order: n d roundings of 2^-53 at most, of a sum of positive terms
    assert abs(got[0] - want) <= n * d * 2.0 ** -53 * want
    assert got == [got[0]] * 4


@pytest.mark.parametrize("n, d", [(32, 524_284), (32, 524_288), (31, 541_201), (29, 578_527), (64, 1_000_003),
                                  (48, 999_999), (48, 1_000_000), (61, 786_432), (61, 786_881), (31, 1_552_673)])
def test_around_the_kernel_of_its_own(n, d):
    """Both sides of 48 M elements and of three workgroups on each compute unit, from which on a kernel behind makes the last sum."""
    X = torch.randn(n, d, device="cuda:0", generator=torch.Generator(device="cuda:0").manual_seed(n))
    want = _reference(X)
    out = torch.full((3,), float("nan"), dtype=torch.float64, device="cuda:0")
    for k in range(3):
        psgd.consensus_dist_async(X, out[k:k + 1])
    got = out.tolist()
    assert abs(got[0] - want) <= n * d * 2.0 ** -53 * want
    assert got == [got[0]] * 3 and psgd.consensus_dist(X) == got[0]


def test_more_launches_than_tickets():
    n = 5
    sizes = [1000, 70_001, 400_000]
    X = [torch.randn(n, d, device="cuda:0") for d in sizes]
    G = [torch.randn(n, d, device="cuda:0") for d in sizes]
    nbr, w = [torch.from_numpy(np.ascontiguousarray(t)).to("cuda:0") for t in psgd.build_mixing(psgd.TOPO_RAND_RING, n, 3, 0)]
    rounds = 3 * TICKETS // len(sizes) + 2
    out = torch.full((rounds, len(sizes)), float("nan"), dtype=torch.float64, device="cuda:0")
    Y = [torch.empty_like(x) for x in X]
    for r in range(rounds):
        for i in range(len(sizes)):
            psgd.mix_step(X[i], Y[i], G[i], nbr, w, 0.1, cdist_out=out[r, i:i + 1])
    for i, y in enumerate(Y):
        want = _reference(y)
        got = out[:, i]
        assert bool((got == got[0]).all())
        assert abs(float(got[0]) - want) <= n * sizes[i] * 2.0 ** -53 * want


def test_graph_replays_between_eager_calls():
    n, d = 6, 300_001
    X, G = torch.randn(n, d, device="cuda:0"), torch.randn(n, d, device="cuda:0")
    Y, Z = torch.empty_like(X), torch.empty_like(X)
    nbr, w = [torch.from_numpy(np.ascontiguousarray(t)).to("cuda:0") for t in psgd.build_mixing(psgd.TOPO_RAND_RING, n, 3, 0)]
    c, e = torch.zeros(1, dtype=torch.float64, device="cuda:0"), torch.zeros(1, dtype=torch.float64, device="cuda:0")
    psgd.mix_step(X, Y, G, nbr, w, 0.1, cdist_out=e)
    want = float(e)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        psgd.mix_step(X, Z, G, nbr, w, 0.1, cdist_out=c)
    for k in range(5):
        c.fill_(float("nan"))
        g.replay()
        e.fill_(float("nan"))
        psgd.mix_step(X, Y, G, nbr, w, 0.1, cdist_out=e)
        torch.cuda.synchronize()
        assert float(c) == want and float(e) == want, k
        assert torch.equal(Y, Z)


def test_graph_with_the_fixed_array_beside_calls_with_the_other():
    """Two arrays of partial sums, hence two streams that may run side by side, one of them a graph:
    over many calls each gets its own distance, also when the launches' workgroup counts differ."""
    gen = torch.Generator(device="cuda:0").manual_seed(3)
    X, G = torch.randn(6, 300_001, device="cuda:0", generator=gen), torch.randn(6, 300_001, device="cuda:0", generator=gen)
    V = torch.randn(3, 500_000, device="cuda:0", generator=gen)
    Y, want_v = torch.empty_like(X), _reference(V)
    nbr, w = [torch.from_numpy(np.ascontiguousarray(t)).to("cuda:0") for t in psgd.build_mixing(psgd.TOPO_RAND_RING, 6, 3, 0)]
    c = torch.zeros(1, dtype=torch.float64, device="cuda:0")
    psgd.mix_step_cd_static(X, Y, G, nbr, w, 0.1, c)
    want = float(c)
    rounds = 2 * TICKETS
    got, got_v = [torch.full((rounds,), float("nan"), dtype=torch.float64, device="cuda:0") for _ in range(2)]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        psgd.mix_step_cd_static(X, Y, G, nbr, w, 0.1, c)
    torch.cuda.synchronize()
    for k in range(rounds):
        with torch.cuda.stream(side):
            g.replay()
            got[k:k + 1].copy_(c)
        psgd.consensus_dist_async(V, got_v[k:k + 1])
    torch.cuda.synchronize()
    assert bool((got == want).all())
    assert bool((got_v == got_v[0]).all()) and abs(float(got_v[0]) - want_v) <= V.numel() * 2.0 ** -53 * want_v


def test_calls_behind_overlapping_ones():
    """Calls of one array of partial sums that run side by side, the caller's mistake: their own distances may be wrong or missing, those of
    later calls in order are right, whichever workgroup counts overlapped."""
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    shapes = [(6, 300_001), (8, 40_000), (6, 300_001), (16, 20_003)]
    data = [[torch.randn(n, d, device="cuda:0", generator=gen) for _ in range(2)] for n, d in shapes]
    data = [(X, torch.empty_like(X), G) for X, G in data]
    tables = [[torch.from_numpy(np.ascontiguousarray(t)).to("cuda:0") for t in psgd.build_mixing(psgd.TOPO_RAND_RING, n, 3, 0)] for n, _ in shapes]
    cd = [torch.zeros(1, dtype=torch.float64, device="cuda:0") for _ in shapes]

    def step(i):
        X, Y, G = data[i]
        psgd.mix_step_cd_static(X, Y, G, *tables[i], 0.1, cd[i])

    want = []
    for i in range(len(shapes)):
        step(i)
        want.append(float(cd[i]))
        assert abs(want[i] - _reference(data[i][1])) <= shapes[i][0] * shapes[i][1] * 2.0 ** -53 * want[i]
    streams = [torch.cuda.Stream() for _ in shapes]
    graphs = []
    for i, s in enumerate(streams):
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[i], stream=s):
            step(i)
    torch.cuda.synchronize()
    for _ in range(60):
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                step(i)
                graphs[i].replay()
    torch.cuda.synchronize()
    for k in range(3):
        for i in range(len(shapes)):
            cd[i].fill_(float("nan"))
            step(i)
            assert float(cd[i]) == want[i], (k, i)
            cd[i].fill_(float("nan"))
            graphs[i].replay()
            assert float(cd[i]) == want[i], (k, i)
