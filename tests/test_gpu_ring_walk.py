"""The ring walk at each depth of its prefetch, from the fewest learners on, with chunks that fill their wavefronts and ones that do not,
workgroups without columns in the last sweep, ragged rows; launches that overlap on several streams and more launches than there are
words for keeping pace.  Every element and the distance against the oracle's sparse form."""
import numpy as np
import pytest

from oracle import psgd_oracle as orc
from paper_2002_01119_amd import inputs as inp

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# n, d, gradients: depth 1 (several sweeps, the last one not for every workgroup), 2, 4 and 6; even and odd counts of rows
CASES = [
    (9, 6_300_004, "f32"), (9, 6_291_459, "bf16"), (15, 6_400_001, "bf16"), (31, 1_180_003, "f32"), (64, 1_966_084, "f32"),
    (65, 990_001, "bf16"), (100, 450_001, "bf16"), (101, 590_000, "f32"), (100, 409_604, "f32"), (128, 330_003, "bf16"),
    (129, 320_000, "f32"), (256, 267_000, "bf16"), (257, 197_001, "f32"), (300, 230_002, "bf16"), (512, 200_000, "f32"),
]


@pytest.fixture(scope="module")
def psgd():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2002_01119_amd import psgd as m
    m.load()
    torch.cuda.set_device(0)
    return m


def _inputs(psgd, n, d, gkind, seed):
    nbr, w = psgd.build_mixing(psgd.TOPO_RAND_RING, n, seed, d)
    X = inp.host_normal_f32((n, d), 1.0, seed) + np.float32(2.0)
    G = inp.host_normal_f32((n, d), 0.5, seed + 1)
    gmax = float(np.abs(G).max()) * 1.01
    if gkind == "bf16":
        G = inp.f32_to_bf16_bits(G)
    # one fp32 rounding per slot and one for the gradient term, each on a partial sum no larger than this
    return X, G, nbr, w, 4 * 2.0 ** -24 * (float(np.abs(X).max()) + 0.2 * gmax)


@pytest.mark.parametrize("n,d,gkind", CASES)
def test_ring_walk_every_element(psgd, n, d, gkind):
    X, G, nbr, w, tol = _inputs(psgd, n, d, gkind, 61 + n)
    want = orc.sparse_mix_step(X, G, nbr, w, 0.2, threads=4)
    Xd = torch.from_numpy(X).to("cuda:0")
    Gd = torch.from_numpy(G.view(np.int16) if gkind == "bf16" else G).to("cuda:0")
    nd, wd = torch.from_numpy(nbr).to("cuda:0"), torch.from_numpy(w).to("cuda:0")
    for form in ("plain", "distance", "in place"):
        Y = torch.full_like(Xd, float("nan")) if form != "in place" else Xd
        c = torch.full((1,), float("nan"), dtype=torch.float64, device="cuda:0") if form != "plain" else None
        psgd.mix_step(Xd, Y, Gd, nd, wd, 0.2, cdist_out=c)
        torch.cuda.synchronize()
        got = Y.cpu().numpy()
        assert np.abs(got - want).max() <= tol, form
        if c is not None:
            ref = orc.sparse_consensus_dist(got.astype(np.float64), threads=4)
            assert abs(c.item() - ref) <= 1e-9 * ref, form
    assert psgd.device_status() == 0


# tables that are not one ring on rows as long: two, three and four rows per lane, rows on and off 128-byte lines
@pytest.mark.parametrize("n,d,gkind", [
    (10, 3_700_003, "f32"), (13, 2_600_000, "bf16"), (16, 1_700_032, "f32"), (17, 1_700_001, "bf16"), (33, 600_001, "f32"),
    (64, 420_032, "bf16"), (100, 350_002, "f32"), (300, 240_032, "bf16"), (301, 240_001, "bf16"), (512, 240_032, "f32")])
def test_other_tables_on_the_same_rows(psgd, n, d, gkind):
    X, G, nbr, w, tol = _inputs(psgd, n, d, gkind, 83 + n)
    rng = np.random.default_rng(n)
    c = rng.random(3).astype(np.float32) + np.float32(0.05)
    nbr = np.stack([rng.permutation(n) for _ in range(3)], axis=1).astype(np.int32)
    w = np.tile((c / c.sum()).astype(np.float32), (n, 1))
    want = orc.sparse_mix_step(X, G, nbr, w, 0.2, threads=4)
    Xd = torch.from_numpy(X).to("cuda:0")
    Gd = torch.from_numpy(G.view(np.int16) if gkind == "bf16" else G).to("cuda:0")
    nd, wd = torch.from_numpy(nbr).to("cuda:0"), torch.from_numpy(w).to("cuda:0")
    for form in ("plain", "distance", "in place"):
        Y = torch.full_like(Xd, float("nan")) if form != "in place" else Xd
        c = torch.full((1,), float("nan"), dtype=torch.float64, device="cuda:0") if form != "plain" else None
        psgd.mix_step(Xd, Y, Gd, nd, wd, 0.2, cdist_out=c)
        torch.cuda.synchronize()
        got = Y.cpu().numpy()
        assert np.abs(got - want).max() <= tol, form
        if c is not None:
            ref = orc.sparse_consensus_dist(got.astype(np.float64), threads=4)
            assert abs(c.item() - ref) <= 1e-9 * ref, form
    bad = nbr.copy()
    bad[n - 1, 2] = n
    before = Xd.clone()
    c = torch.zeros(1, dtype=torch.float64, device="cuda:0")
    psgd.mix_step(Xd, Xd, Gd, torch.from_numpy(bad).to("cuda:0"), wd, 0.2, cdist_out=c)
    torch.cuda.synchronize()
    assert torch.equal(Xd, before) and torch.isnan(c).all() and psgd.device_status() == 1


# global averaging in step: two and four rows on their way, counts of rows that these divide or not, several sweeps, ragged rows
@pytest.mark.parametrize("n,d,gkind", [
    (9, 2_457_600, "f32"), (9, 2_500_003, "bf16"), (16, 819_201, "f32"), (17, 820_002, "bf16"), (31, 1_100_004, "f32"), (33, 600_001, "f32"),
    (48, 310_001, "bf16"), (49, 307_200, "f32"), (50, 590_003, "bf16"), (65, 330_004, "f32"), (130, 307_201, "bf16"), (511, 310_000, "f32")])
def test_global_averaging_every_element(psgd, n, d, gkind):
    X, G, _, _, _ = _inputs(psgd, n, d, gkind, 17 + n)
    g = G if gkind == "f32" else (G.astype(np.uint32) << 16).view(np.float32)
    lr = np.float64(np.float32(0.2))
    mean = X.mean(axis=0, dtype=np.float64)
    # the mean's rounding to fp32 and the last fused operation's, each on a value no larger than this
    tol = 2.0 ** -24 * (2 * float(np.abs(mean).max()) + 0.2 * float(np.abs(g).max()))
    Xd = torch.from_numpy(X).to("cuda:0")
    Gd = torch.from_numpy(G.view(np.int16) if gkind == "bf16" else G).to("cuda:0")
    for form in ("plain", "distance", "in place"):
        Y = torch.full_like(Xd, float("nan")) if form != "in place" else Xd
        c = torch.full((1,), float("nan"), dtype=torch.float64, device="cuda:0") if form != "plain" else None
        psgd.mix_full(Xd, Y, Gd, 0.2, cdist_out=c)
        torch.cuda.synchronize()
        got = Y.cpu().numpy()
        for i in range(0, n, 8):
            assert np.abs(got[i:i + 8] - (mean - lr * g[i:i + 8])).max() <= tol, form
        if c is not None:
            ref = orc.sparse_consensus_dist(got.astype(np.float64), threads=4)
            assert abs(c.item() - ref) <= 1e-9 * ref, form
    assert psgd.device_status() == 0


def test_launches_that_overlap_and_share_pace_words(psgd):
    """Three streams with 100 launches each, so that launches under way at once share words; the bits are those of a launch alone."""
    n, d = 64, 1_000_004
    X, G, nbr, w, _ = _inputs(psgd, n, d, "f32", 7)
    Xd, Gd = torch.from_numpy(X).to("cuda:0"), torch.from_numpy(G).to("cuda:0")
    nd, wd = torch.from_numpy(nbr).to("cuda:0"), torch.from_numpy(w).to("cuda:0")
    alone = torch.empty_like(Xd)
    psgd.mix_step(Xd, alone, Gd, nd, wd, 0.2)
    streams = [torch.cuda.Stream() for _ in range(3)]
    outs = [torch.full_like(Xd, float("nan")) for _ in streams]
    torch.cuda.synchronize()
    for _ in range(100):
        for s, Y in zip(streams, outs):
            psgd.mix_step(Xd, Y, Gd, nd, wd, 0.2, stream=s)
    torch.cuda.synchronize()
    assert all(torch.equal(Y, alone) for Y in outs)
    assert psgd.device_status() == 0
