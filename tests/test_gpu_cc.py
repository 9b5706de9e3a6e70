"""Parity of the HIP connected components (grid mask and CSR) and of the
pointer-jumping entry point with the CPU oracle, bit-exact."""
import itertools
import os

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2409_03771_amd import synth

pytestmark = pytest.mark.gpu
GOLDEN = os.path.join(os.path.dirname(__file__), "golden")


@pytest.fixture(scope="module")
def msc():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2409_03771_amd import msc as m
    return m


def gpu_cc_grid(msc, mask):
    lab = msc.cc_label_grid(torch.from_numpy(np.ascontiguousarray(mask)).cuda())
    torch.cuda.synchronize()
    return lab.cpu().numpy()


def gpu_cc_csr(msc, row_ptr, col, mask=None):
    mt = None if mask is None else torch.from_numpy(mask).cuda()
    lab = msc.cc_label_csr(torch.from_numpy(row_ptr).cuda(),
                           torch.from_numpy(col).cuda(), mt)
    torch.cuda.synchronize()
    return lab.cpu().numpy()


def test_gauss64_threshold_mask(msc):
    f = synth.config_field("gauss64")
    mask = synth.threshold_mask(f, 0.7)
    want, _ = O.cc_grid(mask)
    np.testing.assert_array_equal(gpu_cc_grid(msc, mask), want)


@pytest.mark.parametrize("density", [0.05, 0.3, 0.55, 0.9, 1.0, 0.0])
@pytest.mark.parametrize("dims", [(61, 47, 33), (1, 1, 1), (500, 1, 1),
                                  (1, 70, 60), (80, 90, 1), (129, 3, 2)])
def test_random_masks(msc, dims, density):
    X, Y, Z = dims
    rng = np.random.default_rng(X * 7 + int(density * 100))
    mask = (rng.uniform(size=(Z, Y, X)) < density).astype(np.uint8)
    want, _ = O.cc_grid(mask)
    np.testing.assert_array_equal(gpu_cc_grid(msc, mask), want)


def test_every_mask_3x3x2_in_one_call(msc):
    """All 2^18 masks of a 3x3x2 grid stacked along z with an empty plane
    between them: one call labels every mask independently."""
    M = np.array(list(itertools.product((0, 1), repeat=18)), np.uint8)
    big = np.zeros((M.shape[0], 3, 3, 3), np.uint8)
    big[:, :2] = M.reshape(-1, 2, 3, 3)
    big = big.reshape(-1, 3, 3)
    want, _ = O.cc_grid(big)
    np.testing.assert_array_equal(gpu_cc_grid(msc, big), want)


def test_gaussian_mask_ragged(msc):
    f = synth.gaussian_field((190, 171, 93), 60, seed=5)
    for q in (0.1, 0.5, 0.7, 0.9):
        mask = synth.threshold_mask(f, q)
        want, _ = O.cc_grid(mask)
        np.testing.assert_array_equal(gpu_cc_grid(msc, mask), want, str(q))


@pytest.fixture(scope="module")
def kuhn():
    return synth.kuhn_csr(28, seed=2, nbumps=10)


def test_csr_masked_explicit_and_full(msc, kuhn):
    g = kuhn
    want, _ = O.cc_csr(g["row_ptr"], g["col_idx"], g["mask"])
    np.testing.assert_array_equal(
        gpu_cc_csr(msc, g["row_ptr"], g["col_idx"], g["mask"]), want)
    want, _ = O.cc_csr(g["fg_row_ptr"], g["fg_col_idx"])
    np.testing.assert_array_equal(
        gpu_cc_csr(msc, g["fg_row_ptr"], g["fg_col_idx"]), want)
    got = gpu_cc_csr(msc, g["row_ptr"], g["col_idx"])
    assert (got == 0).all()


@pytest.mark.parametrize("seed", [0, 1, 2, 3])
def test_csr_random_graph_one_sided(msc, seed):
    """Random sparse graph listed one-sided (each edge in one row only)."""
    rng = np.random.default_rng(seed)
    n = 20000
    E = rng.integers(0, n, size=(int(n * (0.3 + 0.3 * seed)), 2))
    E = np.sort(E, axis=1)
    order = np.lexsort((E[:, 1], E[:, 0]))
    E = E[order]
    row_ptr = np.zeros(n + 1, np.int64)
    np.add.at(row_ptr, E[:, 0] + 1, 1)
    row_ptr = np.cumsum(row_ptr)
    col = E[:, 1].astype(np.int32)
    want, _ = O.cc_csr(row_ptr, col)
    np.testing.assert_array_equal(gpu_cc_csr(msc, row_ptr, col), want)
    mask = (rng.uniform(size=n) < 0.7).astype(np.uint8)
    want, _ = O.cc_csr(row_ptr, col, mask)
    np.testing.assert_array_equal(gpu_cc_csr(msc, row_ptr, col, mask), want)


def test_csr_edge_cases(msc):
    # no edges at all
    n = 1000
    rp = np.zeros(n + 1, np.int64)
    col = np.zeros(0, np.int32)
    lab = msc.cc_label_csr(torch.from_numpy(rp).cuda(),
                           torch.empty(0, dtype=torch.int32, device="cuda"))
    assert (lab.cpu().numpy() == np.arange(n)).all()
    # a long path listed in decreasing order: worst case for hooking by id
    n = 5000
    perm = np.random.default_rng(3).permutation(n)
    rows = [[] for _ in range(n)]
    for i in range(n - 1):
        a, b = perm[i], perm[i + 1]
        rows[a].append(b)
        rows[b].append(a)
    rp = np.zeros(n + 1, np.int64)
    rp[1:] = np.cumsum([len(r) for r in rows])
    col = np.array([u for r in rows for u in sorted(r)], np.int32)
    assert (gpu_cc_csr(msc, rp, col) == 0).all()
    # out-of-range column index is rejected
    bad = col.copy()
    bad[17] = n + 5
    with pytest.raises(msc.MscError) as e:
        gpu_cc_csr(msc, rp, bad)
    assert e.value.code == msc.MSC_EINVAL


def _fig2_rows():
    rows = {}
    with open(os.path.join(GOLDEN, "fig2_pointer_table.txt")) as fh:
        for line in fh:
            if line.startswith("#") or not line.strip():
                continue
            p = line.split()
            rows[p[0]] = p[1:]
    return rows


def test_pointer_jump_reproduces_fig2(msc):
    rows = _fig2_rows()
    L = {c: i for i, c in enumerate("ABCDEFGHIJKLMNOP")}
    d0 = np.arange(16, dtype=np.int64)
    for c in "ABCDEFGHIJKLMNO":
        d0[L[c]] = L[rows[c][0]] if c in rows else L[c] + 1
    for r in (1, 2, 3):
        d = torch.from_numpy(d0).cuda()
        msc.pointer_jump(d, rounds=r, synchronous=True)
        got = d.cpu().numpy()
        for c, cols in rows.items():
            want = "P" if cols[r] == "-" else cols[r]
            assert got[L[c]] == L[want], (c, r)
    d = torch.from_numpy(d0).cuda()
    msc.pointer_jump(d)             # in place, to convergence
    assert (d.cpu().numpy() == 15).all()


def test_pointer_jump_random_forest(msc):
    rng = np.random.default_rng(9)
    n = 1 << 20
    parent = np.arange(n, dtype=np.int64)
    # random forest: each vertex points to a smaller id or itself
    nonroot = rng.uniform(size=n) < 0.999
    parent[nonroot] = (rng.uniform(size=nonroot.sum()) *
                       np.arange(n)[nonroot]).astype(np.int64)
    want = O.sync_doubling(parent, 25)
    for sync in (True, False):
        d = torch.from_numpy(parent).cuda()
        msc.pointer_jump(d, synchronous=sync)
        np.testing.assert_array_equal(d.cpu().numpy(), want)


def test_batched_masks_equal_oracle(msc):
    """70 masks of uneven shapes (more than one launch's worth, with edge
    shapes and empty and full masks) in one batched call: every mask's
    labels equal the oracle's, ids local to the mask."""
    rng = np.random.default_rng(31)
    masks = []
    shapes = [(1, 1, 1), (33, 17, 17), (64, 1, 1), (1, 40, 3), (32, 16, 16)]
    for k in range(70):
        dims = shapes[k] if k < len(shapes) else tuple(
            int(x) for x in rng.integers(1, 70, size=3))
        X, Y, Z = dims
        if k == 5:
            m = np.zeros((Z, Y, X), np.uint8)
        elif k == 6:
            m = np.ones((Z, Y, X), np.uint8)
        elif k % 3 == 0:
            f = synth.gaussian_field(dims, 6, 300 + k)
            m = synth.threshold_mask(f, 0.6)
        else:
            m = (rng.uniform(size=(Z, Y, X)) < rng.uniform(0.1, 0.9)).astype(
                np.uint8)
        masks.append(m)
    dev = [torch.from_numpy(m).cuda() for m in masks]
    labels = [torch.full((m.size,), -7, dtype=torch.int64, device="cuda")
              for m in masks]
    msc.cc_label_grid_batched_into(dev, labels)
    torch.cuda.synchronize()
    for k, (m, lab) in enumerate(zip(masks, labels)):
        want, _ = O.cc_grid(m)
        np.testing.assert_array_equal(lab.cpu().numpy(), want,
                                      err_msg=f"mask {k} {m.shape}")


def test_batched_masks_edge_cases(msc):
    assert msc.cc_label_grid_batched([]) == []
    m = torch.ones((5, 4, 3), dtype=torch.uint8, device="cuda")
    with pytest.raises(TypeError):
        msc.cc_label_grid_batched_into([m], [torch.empty(60, dtype=torch.int32,
                                                         device="cuda")])
    with pytest.raises(ValueError):
        msc.cc_label_grid_batched_into([m], [torch.empty(59, dtype=torch.int64,
                                                         device="cuda")])
    (lab,) = msc.cc_label_grid_batched([m])
    torch.cuda.synchronize()
    assert (lab == 0).all()


@pytest.mark.parametrize("n", [1, 2, 3, 63, 65, 4095, 4096, 4097, 8191, 8192,
                               8193, 100003])
@pytest.mark.parametrize("deg", [0.6, 2.5])
@pytest.mark.parametrize("both", [False, True])
def test_csr_sizes(msc, n, deg, both):
    """Random graphs around the sizes where the passes change, without and
    with a large component, each edge listed once or twice, in no order, with
    self-loops; unmasked, half masked and nearly unmasked."""
    rng = np.random.default_rng(n + int(10 * deg))
    E = rng.integers(0, n, size=(int(n * deg), 2))
    if both:
        E = np.concatenate([E, E[:, ::-1]])
    E = E[rng.permutation(len(E))]
    order = np.argsort(E[:, 0], kind="stable")
    row_ptr = np.zeros(n + 1, np.int64)
    row_ptr[1:] = np.cumsum(np.bincount(E[:, 0], minlength=n))
    col = np.ascontiguousarray(E[order, 1].astype(np.int32))
    for share in (None, 0.5, 0.01):
        mask = None if share is None else (
            rng.uniform(size=n) < share).astype(np.uint8)
        want, _ = O.cc_csr(row_ptr, col, mask)
        np.testing.assert_array_equal(
            gpu_cc_csr(msc, row_ptr, col, mask), want, err_msg=str(share))
    if col.size:
        col[col.size // 2] = n
        with pytest.raises(msc.MscError) as e:
            gpu_cc_csr(msc, row_ptr, col)
        assert e.value.code == msc.MSC_EINVAL


@pytest.mark.parametrize("dims", [(31, 17, 16), (32, 16, 17), (33, 15, 33),
                                  (64, 33, 16), (65, 32, 18), (97, 1, 1),
                                  (1, 40, 35), (2, 18, 34), (130, 50, 1)])
@pytest.mark.parametrize("kind", [0.1, 0.35, 0.6, 0.95, "comb", "full"])
def test_rows_and_runs(msc, dims, kind):
    """Around the 32 x 16 x 16 of a tile: masks of every density, the most runs
    a row can hold, and a full one, at a byte address of no alignment; also
    through the entry point without a context and through slabs."""
    X, Y, Z = dims
    rng = np.random.default_rng(sum(dims))
    if kind == "comb":
        x, y, z = np.meshgrid(np.arange(X), np.arange(Y), np.arange(Z),
                              indexing="ij")
        mask = ((x + 3 * y + 5 * z) % 2 == 0).transpose(2, 1, 0)
        mask = mask & (rng.uniform(size=mask.shape) < 0.98)
    elif kind == "full":
        mask = np.ones((Z, Y, X), bool)
    else:
        mask = rng.uniform(size=(Z, Y, X)) < kind
    # any non-zero byte is a feature
    mask = mask.astype(np.uint8) * rng.choice([1, 2, 128, 255], size=mask.shape
                                              ).astype(np.uint8)
    want, _ = O.cc_grid(mask)
    for shift in (0, 1, 7):
        buf = torch.empty(mask.size + shift, dtype=torch.uint8, device="cuda")
        part = buf[shift:]
        part.copy_(torch.from_numpy(mask.reshape(-1)))
        lab = torch.empty(mask.size, dtype=torch.int64, device="cuda")
        msc.cc_label_grid_into(part, lab, dims=dims)
        np.testing.assert_array_equal(lab.cpu().numpy(), want, err_msg=str(shift))
    lab.zero_()
    msc.cc_label_grid_noalloc_into(part, lab, dims=dims)
    np.testing.assert_array_equal(lab.cpu().numpy(), want, err_msg="noalloc")
    for ranks in {1, min(2, Z), min(5, Z)}:
        got = msc.cc_label_grid_ranks(part, ranks, dims=dims)
        np.testing.assert_array_equal(got.cpu().numpy(), want,
                                      err_msg=f"{ranks} ranks")


@pytest.mark.parametrize("n", [4095, 4096, 8193, 70_000, 1 << 20,
                               (1 << 21) + 5])
@pytest.mark.parametrize("order", ["rising", "swapped", "interleaved",
                                   "random"])
def test_csr_curves(msc, n, order):
    """Curves, whose hooks and joins can form one chain through half of the
    vertices (ids that rise along it), whole and cut into pieces by the mask.
    At a million vertices a call takes 0.2 to 0.35 ms; walking those chains
    link by link takes 8 ms and more."""
    i = np.arange(n)
    ids = {"rising": i, "swapped": np.where(i ^ 1 < n, i ^ 1, i),
           "interleaved": np.where(i % 2 == 0, i // 2, (n + 1) // 2 + i // 2),
           "random": np.random.default_rng(n).permutation(n)}[order]
    pos = np.empty(n, np.int64)
    pos[ids] = i
    nb = np.stack([np.where(pos > 0, ids[np.maximum(pos - 1, 0)], -1),
                   np.where(pos < n - 1, ids[np.minimum(pos + 1, n - 1)], -1)],
                  1)
    nb.sort(axis=1)
    rp = np.zeros(n + 1, np.int64)
    rp[1:] = np.cumsum((nb >= 0).sum(1))
    g = [torch.from_numpy(a).cuda()
         for a in (rp, nb[nb >= 0].astype(np.int32))]
    for cut in (None, n // 3 + 1, 5):
        mask = None
        starts = np.zeros(1, np.int64)
        inside = np.ones(n, bool)  # along the curve
        if cut is not None:
            inside = i % cut != cut - 1
            mask = np.empty(n, np.uint8)
            mask[ids] = inside
            mask = torch.from_numpy(mask).cuda()
            starts = np.arange(0, n, cut)
        least = np.minimum.reduceat(np.where(inside, ids, n), starts)
        want = np.empty(n, np.int64)
        want[ids] = np.where(inside, least[np.searchsorted(starts, i, "right") - 1], -1)
        ms = []
        for _ in range(4):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            got = msc.cc_label_csr(*g, mask)
            b.record()
            b.synchronize()
            ms.append(a.elapsed_time(b))
        np.testing.assert_array_equal(got.cpu().numpy(), want, err_msg=f"{cut}")
        if n == 1 << 20:
            assert min(ms) < 4.0, (cut, ms)


@pytest.mark.parametrize("dims", [(64, 48, 33), (131, 70, 1), (33, 17, 50)])
@pytest.mark.parametrize("kind", ["comb", "teeth", "checker", "stairs", "dots"])
def test_rows_of_many_runs(msc, dims, kind):
    """Masks whose rows hold up to 16 runs of a tile's 32 columns, which touch
    one long run, a run each, or only diagonally."""
    X, Y, Z = dims
    z, y, x = np.ogrid[:Z, :Y, :X]
    m = {"comb": (x % 2 == 0) | (y % 16 == 5),
         "teeth": (x % 3 != 1) & ((x % 2 == 0) | (y % 5 == 0) | (z % 4 == 2)),
         "checker": (x + y + z) % 2 == 0,
         "stairs": ((x + y) % 4 == 0) | ((x - z) % 5 == 0),
         "dots": (x % 2 == 0) & (y % 2 == 0) & (z % 2 == 0)}[kind]
    m = np.ascontiguousarray(np.broadcast_to(m, (Z, Y, X))).astype(np.uint8)
    want, _ = O.cc_grid(m)
    got = msc.cc_label_grid(torch.from_numpy(m).cuda())
    np.testing.assert_array_equal(got.cpu().numpy(), want)


@pytest.mark.parametrize("n", [1 << 14, (1 << 14) + 1, 1 << 17, (1 << 17) + 1])
@pytest.mark.parametrize("deg", [1, 4])
def test_csr_sizes_of_shared_launches(msc, n, deg):
    """On both sides of where the rounds of joins share a launch and where
    every block finds the tree to mark, sparse (many small trees) and dense."""
    rng = np.random.default_rng(n + deg)
    rp = np.arange(n + 1, dtype=np.int64) * deg
    col = rng.integers(0, n, size=n * deg).astype(np.int32)
    for mask in (None, (rng.random(n) < 0.6).astype(np.uint8)):
        want, _ = O.cc_csr(rp, col, mask)
        np.testing.assert_array_equal(gpu_cc_csr(msc, rp, col, mask), want)
    bad = col.copy()
    bad[-1] = n
    with pytest.raises(msc.MscError):
        gpu_cc_csr(msc, rp, bad)
