"""Critical points (link components) and the extremum graph through the C
ABI, bit-exact against the oracle: random fields with ties on 3-D, 2-D and
1-D grids, Gaussian and Perlin fields; and at 1024^3, sampled vertices
against the oracle on their neighbourhood box plus whole-field counts."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2409_03771_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def msc():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2409_03771_amd import msc as m
    return m


def check(msc, f, tag):
    t = torch.from_numpy(np.ascontiguousarray(f)).cuda()
    code = msc.critical_points(t).cpu().numpy()
    lc, uc, _ = O.critical(f)
    np.testing.assert_array_equal(code & 15, lc, err_msg=f"{tag} lower")
    np.testing.assert_array_equal(code >> 4, uc, err_msg=f"{tag} upper")
    a, d, _ = msc.segment(t)
    E = msc.extremum_graph(t, a, d).cpu().numpy()
    torch.cuda.synchronize()
    W = O.extremum_edges(f, a.cpu().numpy(), d.cpu().numpy())
    np.testing.assert_array_equal(E, W, err_msg=f"{tag} extremum graph")
    return code, E


@pytest.mark.parametrize("dims", [(23, 19, 17), (40, 33, 1), (1, 29, 31),
                                  (50, 1, 1), (1, 1, 1), (2, 2, 2),
                                  (65, 3, 2)])
@pytest.mark.parametrize("levels", [None, 2])
def test_random_fields(msc, dims, levels):
    f = synth.random_field(dims, seed=sum(dims) * 3 + (levels or 0),
                           levels=levels)
    check(msc, f, f"{dims} levels={levels}")


def test_gaussian_and_perlin(msc):
    code, E = check(msc, synth.config_field("gauss64"), "gauss64")
    assert (E[:, 2] == 1).any() and (E[:, 2] == -1).any()
    check(msc, synth.perlin_field((70, 60, 50), seed=5), "perlin")


def test_nan_is_reported(msc):
    f = np.zeros((4, 4, 4), np.float32)
    f[2, 1, 3] = np.nan
    with pytest.raises(Exception):
        msc.critical_points(torch.from_numpy(f).cuda())


def test_fullsize_sampled(msc):
    """gauss1024: link codes of 3000 random vertices equal the oracle's on
    the vertex's neighbourhood box (the link only sees the neighbours, and a
    sub-box keeps the id order); extremum counts equal the segmentation's;
    every ascending edge ends at a maximum, one per upper-link component."""
    print("[critical] gauss1024", flush=True)
    f = synth.config_field("gauss1024", device="cuda")
    code = msc.critical_points(f)
    a, d, _ = msc.segment(f, want=("asc", "desc"))
    st = msc.last_stats()
    E = msc.extremum_graph(f, a, d)
    torch.cuda.synchronize()
    assert int((code >> 4 == 0).sum()) == st["n_maxima"]
    assert int((code & 15 == 0).sum()) == st["n_minima"]
    lc = (code & 15).long()
    uc = (code >> 4).long()
    want = int(torch.where(uc >= 2, uc, 0).sum() + torch.where(lc >= 2, lc, 0).sum())
    assert E.shape[0] == want
    up = E[E[:, 2] == 1]
    assert bool((a[up[:, 1].long()] == up[:, 1]).all())
    dn = E[E[:, 2] == -1]
    assert bool((d[dn[:, 1].long()] == dn[:, 1]).all())
    fh = f.cpu().numpy()
    ch = code.cpu().numpy()
    rng = np.random.default_rng(0)
    n = 1024
    for v in rng.integers(0, n ** 3, size=3000):
        x, y, z = v % n, (v // n) % n, v // (n * n)
        x0, y0, z0 = max(x - 1, 0), max(y - 1, 0), max(z - 1, 0)
        box = np.ascontiguousarray(fh[z0:z + 2, y0:y + 2, x0:x + 2])
        bl, bu, _ = O.critical(box)
        bx, by = box.shape[2], box.shape[1]
        k = (x - x0) + bx * (y - y0) + bx * by * (z - z0)
        assert (ch[v] & 15, ch[v] >> 4) == (bl[k], bu[k]), int(v)


@pytest.mark.parametrize("dims", [(64, 1, 9), (8, 8, 17), (7, 9, 21),
                                  (63, 5, 3), (65, 16, 2), (513, 1, 5),
                                  (1, 1, 300), (20, 26, 33), (300, 200, 1)])
@pytest.mark.parametrize("kind", ["noise", "smooth"])
def test_runs_and_walks(msc, dims, kind):
    """Around the 64 positions of a run, the 512 of a block and the planes of
    a walk, planes narrower than a run, with nearly every vertex marked and
    with few; and again from a workspace without room for the marks."""
    f = (synth.random_field(dims, seed=9) if kind == "noise" else
         synth.perlin_field(dims, seed=9, frequency=0.15))
    _, E = check(msc, f, f"{dims} {kind}")
    t = torch.from_numpy(np.ascontiguousarray(f)).cuda()
    a, d, _ = msc.segment(t)
    torch.cuda.synchronize()
    nb = (f.size + 255) // 256
    small = torch.empty(4 * nb + 8 * (nb + 1) + 8192, dtype=torch.uint8,
                        device="cuda")
    try:
        msc.set_workspace(small)
        again = msc.extremum_graph(t, a, d).cpu().numpy()
    finally:
        msc.set_workspace(None)
    np.testing.assert_array_equal(again, E, err_msg=f"{dims} small workspace")


@pytest.mark.parametrize("dims", [(191, 1, 6), (192, 1, 6), (193, 1, 6),
                                  (12, 16, 33), (16, 12, 1), (300, 200, 2),
                                  (15, 1, 70), (1, 3, 200)])
@pytest.mark.parametrize("levels", [None, 3])
def test_walks_and_single_vertices(msc, dims, levels):
    """On both sides of where planes are walked: their width and number."""
    f = synth.random_field(dims, seed=sum(dims), levels=levels)
    check(msc, f, f"{dims} levels={levels}")


def test_longest_chain(msc):
    """A chain of vertices along z, longer than a launch has blocks for where a
    block takes 16 planes."""
    n = (1 << 27) + 37
    print(f"[critical] 1x1x{n}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(1)
    f = torch.randint(0, 50, (n,), generator=g, device="cuda").float()
    code = msc.critical_points(f.reshape(n, 1, 1))
    low = torch.zeros(n, dtype=torch.uint8, device="cuda")
    low[1:] += f[:-1] <= f[1:]   # the neighbour of smaller id: below when equal
    low[:-1] += f[1:] < f[:-1]
    here = torch.full((n,), 2, dtype=torch.uint8, device="cuda")
    here[0] = here[-1] = 1
    assert torch.equal(code, low | (here - low) << 4)


@pytest.mark.parametrize("dims", [(128, 128, 130), (96, 90, 70), (300, 200, 40)])
@pytest.mark.parametrize("kind", ["noise", "mixed", "smooth", "smoother"])
def test_runs_per_wave(msc, dims, kind):
    """Grids of enough runs for a wave to take 1, 2, 4, 8 and more of them, with
    marks everywhere, in a part of the planes, and sparse: the marked walk's
    edges equal those of the pass over blocks of 256 vertices."""
    X, Y, Z = dims
    f = synth.perlin_field(dims, seed=5,
                           frequency=0.02 if kind == "smoother" else 0.1)
    if kind in ("noise", "mixed"):
        rough = synth.random_field(dims, seed=6)
        f = np.where(np.arange(Z)[:, None, None] % 16 <
                     (16 if kind == "noise" else 2), rough, f)
    f = f.astype(np.float32)
    t = torch.from_numpy(np.ascontiguousarray(f)).cuda()
    a, d, _ = msc.segment(t)
    got = msc.extremum_graph(t, a, d)
    nb = (f.size + 255) // 256
    small = torch.empty(4 * nb + 8 * (nb + 1) + 8192, dtype=torch.uint8,
                        device="cuda")
    small = small[(-small.data_ptr()) % 256:]
    msc.set_workspace(small)
    try:
        want = msc.extremum_graph(t, a, d)
    finally:
        msc.set_workspace(None)
    assert got.shape[0] > 0
    assert torch.equal(got, want)


def test_noise_costs_no_more_than_the_dense_pass(msc):
    """A graph of pure noise takes no longer from the marked vertices than from
    the pass that looks at every vertex (which a workspace without room for
    the marks gets); it took 1.4 times as long when a run was listed by one
    lane."""
    t = torch.from_numpy(synth.random_field((256, 240, 200), seed=8)).cuda()
    a, d, _ = msc.segment(t)
    n = msc.extremum_graph(t, a, d).shape[0]
    edges = torch.empty((n, 3), dtype=torch.int32, device="cuda")
    nb = (t.numel() + 255) // 256
    small = torch.empty(4 * nb + 8 * (nb + 1) + 8192, dtype=torch.uint8,
                        device="cuda")

    def best():
        ms = []
        for _ in range(8):
            x, y = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            x.record()
            assert msc.extremum_graph_into(t, a, d, edges) == n
            y.record()
            y.synchronize()
            ms.append(x.elapsed_time(y))
        return min(ms)

    marked = best()
    msc.set_workspace(small[(-small.data_ptr()) % 256:])
    try:
        dense = best()
    finally:
        msc.set_workspace(None)
    assert marked < 1.2 * dense, (marked, dense)
