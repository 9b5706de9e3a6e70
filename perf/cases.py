"""Work that users of this framework have it do, through its public entry
points: inputs, one pass, and the bytes a pass cannot do without.

A case is a dict of plain values; ``kind`` names the entry point and the rest
its sizes and options.  Every input is made on the GPU from the seed alone.
Fields are the two kinds of the package's own workloads: sums of Gaussian
bumps with a little noise ("gauss": smooth near the bumps, noise far from
them) and one layer of Perlin noise ("perlin": many small cells); masks are
those fields above a quantile.  All outputs are ids or codes (whole numbers),
so a pass either gives the same values or is wrong.
"""
from __future__ import annotations

import math

import torch

from paper_2409_03771_amd import msc, synth

DEVICE = "cuda:0"
ALL = "asc,desc,ms"


def listed():
    return [
        # The smallest ordinary call: one 64^3 field, outputs allocated and
        # the device's verdict awaited by the call, as interactive use does.
        dict(name="segment_64", kind="segment", x=64, y=64, z=64,
             field="gauss", bumps=8, want=ALL, check=True),
        # A field of odd sides from a time step or a subvolume, cells only
        # (the outcome is checked later, as a pipeline does).
        dict(name="segment_ragged_ms", kind="segment", x=223, y=157, z=101,
             field="gauss", bumps=24, want="ms", check=False),
        # The paper's synthetic workload at its smaller size: 0.9M cells.
        dict(name="segment_perlin512", kind="segment", x=512, y=512, z=512,
             field="perlin", bumps=0, want=ALL, check=False),
        # The headline size, a billion vertices.
        dict(name="segment_gauss1024", kind="segment", x=1024, y=1024, z=1024,
             field="gauss", bumps=512, want=ALL, check=False),
        # Many fields of uneven shapes in one call (a service's queue, an
        # ensemble): the recipe of the batch workload, a quarter of its count.
        dict(name="batch_64", kind="batch", count=64, lo=32, hi=256, shapes=3,
             want=ALL),
        # A time series with fixed buffers: the captured graph replayed on
        # whatever the buffers hold.
        dict(name="graph_series", kind="graph", count=4, lo=64, hi=128,
             shapes=11, want=ALL),
        # Components of a small odd-sided mask, half of it feature (the
        # threshold study's middle level).
        dict(name="cc_ragged", kind="cc", x=245, y=190, z=133,
             field="perlin", bumps=0, quantile=0.5),
        # Components of a billion-vertex mask, the top 30 %.
        dict(name="cc_gauss1024", kind="cc", x=1024, y=1024, z=1024,
             field="gauss", bumps=512, quantile=0.7),
        # Components of a feature mask on a tetrahedral mesh's vertices
        # (50M vertices, 694M entries, ids in no order).
        dict(name="cc_csr_368", kind="cc_csr", axis=368, bumps=24,
             quantile=0.7),
        # Segmentation of a field on such a mesh.
        dict(name="segment_csr_208", kind="segment_csr", axis=208, bumps=16,
             want=ALL),
        # The adjacency of a mesh from its tetrahedra (24M of them).
        dict(name="tets_160", kind="tets", axis=160),
        # What follows a segmentation: critical points and extremum graph.
        dict(name="topology_512", kind="topology", x=512, y=512, z=512,
             field="perlin", bumps=0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid(rng, lo, hi, top):
    """Three sides, each over the logarithm of [lo, hi], at most `top`
    vertices together; one grid in eight is a plane."""
    while True:
        x, y, z = (_log(rng, lo, hi) for _ in range(3))
        if rng.random() < 0.125:
            x, y, z = 4 * x, 4 * y, 1
        if x * y * z <= top:
            return dict(x=x, y=y, z=z)


def _field(rng):
    field = rng.choice(["gauss", "perlin"])
    return dict(field=field, bumps=_log(rng, 8, 128) if field == "gauss" else 0)


def draw(rng):
    kind = rng.choice(["segment", "segment", "segment", "batch", "graph", "cc",
                       "cc", "cc_csr", "segment_csr", "tets", "topology"])
    want = rng.choice([ALL, ALL, "ms", "asc,desc"])
    if kind == "segment":
        return dict(kind=kind, **_grid(rng, 24, 800, 1 << 28), **_field(rng),
                    want=want, check=rng.random() < 0.3)
    if kind == "batch":
        lo = _log(rng, 16, 64)
        return dict(kind=kind, count=_log(rng, 3, 96), lo=lo,
                    hi=_log(rng, 2 * lo, 256), shapes=rng.randrange(1, 10000),
                    want=want)
    if kind == "graph":
        lo = _log(rng, 16, 96)
        return dict(kind=kind, count=_log(rng, 1, 12), lo=lo,
                    hi=_log(rng, lo + 1, 192), shapes=rng.randrange(1, 10000),
                    want=want)
    if kind == "cc":
        return dict(kind=kind, **_grid(rng, 24, 800, 1 << 28), **_field(rng),
                    quantile=rng.choice([0.1, 0.5, 0.7, 0.9, 0.999]))
    if kind == "cc_csr":
        return dict(kind=kind, axis=_log(rng, 16, 320), bumps=_log(rng, 4, 32),
                    quantile=rng.choice([0.0, 0.3, 0.7, 0.9]))
    if kind == "segment_csr":
        return dict(kind=kind, axis=_log(rng, 16, 208), bumps=_log(rng, 4, 32),
                    want=want)
    if kind == "tets":
        return dict(kind=kind, axis=_log(rng, 8, 160))
    return dict(kind=kind, **_grid(rng, 24, 512, 1 << 27), **_field(rng))


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------


def _make_field(dims, field, bumps, seed):
    """float32 [Z, Y, X] on the GPU."""
    if field == "perlin":
        chunk = max(1, (1 << 25) // max(1, dims[0] * dims[1]))
        return synth.perlin_field(dims, seed, device=DEVICE, z_chunk=chunk)
    f = synth.gaussian_field(dims, bumps, seed, noise=False, device=DEVICE)
    g = torch.Generator(device=DEVICE).manual_seed(seed)
    noise = torch.rand(f.shape, generator=g, device=DEVICE)
    return f.add_(noise.mul_(2 * synth.NOISE).sub_(synth.NOISE))


def _make_mask(f, quantile):
    """uint8, about 1 - quantile of it set (the quantile of a sample)."""
    flat = f.reshape(-1)
    sample = flat[::max(1, flat.numel() >> 22)].sort().values
    k = min(int(quantile * sample.numel()), sample.numel() - 1)
    if quantile == 0.0:
        return torch.ones_like(f, dtype=torch.uint8)
    return (f > sample[k]).to(torch.uint8)


_EDGES = [(1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 1, 0), (1, 0, 1), (0, 1, 1),
          (1, 1, 1)]


def _mesh_csr(n, seed):
    """Adjacency of the Kuhn tetrahedralisation of n^3 vertices whose ids are
    a random permutation (rows in increasing order), and that permutation
    (grid vertex -> id)."""
    g = torch.Generator(device=DEVICE).manual_seed(seed)
    n3 = n ** 3
    perm = torch.randperm(n3, generator=g, device=DEVICE)
    inv = torch.empty_like(perm)
    inv[perm] = torch.arange(n3, device=DEVICE)
    small = perm.to(torch.int32)
    x, y, z = inv % n, (inv // n) % n, inv // (n * n)
    none = 2 ** 31 - 1
    cols = []
    for s in (1, -1):
        for dx, dy, dz in _EDGES:
            ok = torch.ones(n3, dtype=torch.bool, device=DEVICE)
            for c, d in ((x, s * dx), (y, s * dy), (z, s * dz)):
                if d:
                    ok &= (c + d >= 0) & (c + d < n)
            to = inv + s * (dx + n * dy + n * n * dz)
            cols.append(torch.where(ok, small[to.clamp_(0, n3 - 1)], none))
    del x, y, z, inv, small
    # Each row's 14 entries sorted by a transposition network, absent last.
    for r in range(len(cols)):
        for i in range(r & 1, len(cols) - 1, 2):
            cols[i], cols[i + 1] = (torch.minimum(cols[i], cols[i + 1]),
                                    torch.maximum(cols[i], cols[i + 1]))
    nbr = torch.stack(cols, 1)
    del cols
    valid = nbr != none
    row_ptr = torch.zeros(n3 + 1, dtype=torch.int64, device=DEVICE)
    torch.cumsum(valid.sum(1), 0, out=row_ptr[1:])
    return row_ptr, nbr[valid], perm


def _mesh_field(n, bumps, seed, perm):
    """A smooth field on the mesh's vertices, in id order."""
    f = synth.gaussian_field((n, n, n), bumps, seed, noise=False,
                             device=DEVICE).reshape(-1)
    out = torch.empty_like(f)
    out[perm] = f
    return out


def _mesh_tets(n, seed):
    """int32 [6 (n-1)^3, 4]: the Kuhn tetrahedra in the order of their cubes,
    with permuted vertex ids."""
    g = torch.Generator(device=DEVICE).manual_seed(seed)
    perm = torch.randperm(n ** 3, generator=g, device=DEVICE).to(torch.int32)
    a = torch.arange(n - 1, device=DEVICE)
    base = (a[None, None, :] + n * a[None, :, None] +
            n * n * a[:, None, None]).reshape(-1)
    step = (1, n, n * n)
    off = [[0, step[i], step[i] + step[j], 1 + n + n * n]
           for i in range(3) for j in range(3) if i != j]
    off = torch.tensor(off, device=DEVICE)
    out = torch.empty((base.numel(), 6, 4), dtype=torch.int32, device=DEVICE)
    for k in range(6):
        for c in range(4):
            out[:, k, c] = perm[base + off[k, c]]
    return out.reshape(-1, 4)


def _specs(case):
    """Shapes and bump counts of a batch: the same for every seed."""
    return [(d, nb) for d, nb, _ in synth.batch_specs(
        case["count"], seed=case["shapes"], lo=case["lo"], hi=case["hi"])]


def _outputs(sizes, want):
    """One int32 buffer per wanted output, and its part for every field
    (each field's part starts on a 256-byte boundary)."""
    at, total = [], 0
    for n in sizes:
        at.append(total)
        total += (n + 63) // 64 * 64
    bufs = {k: torch.zeros(total, dtype=torch.int32, device=DEVICE)
            for k in want}
    parts = [tuple(bufs[k][a:a + n] if k in bufs else None
                   for k in ("asc", "desc", "ms")) for a, n in zip(at, sizes)]
    return bufs, parts


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case, want=tuple(case.get("want", "").split(",")))
    if kind in ("segment", "cc", "topology"):
        dims = (case["x"], case["y"], case["z"])
        f = _make_field(dims, case["field"], case["bumps"], seed)
    if kind == "segment":
        s["field"] = f
        if not case["check"]:
            s["bufs"], (s["out"],) = _outputs([f.numel()], s["want"])
    elif kind in ("batch", "graph"):
        specs = _specs(case)
        s["fields"] = [_make_field(d, "gauss", nb, 1000 * seed + i)
                       for i, (d, nb) in enumerate(specs)]
        s["bufs"], s["outs"] = _outputs([f.numel() for f in s["fields"]],
                                        s["want"])
        if kind == "graph":
            s["graph"] = msc.Graph(s["fields"], s["outs"])
    elif kind == "cc":
        s["mask"] = _make_mask(f, case["quantile"])
        s["labels"] = torch.empty(f.numel(), dtype=torch.int64, device=DEVICE)
    elif kind == "topology":
        s["field"] = f
        s["asc"], s["desc"], _ = msc.segment(f, want=("asc", "desc"))
        # Room for two edges per vertex, which noise does not reach.
        s["edges"] = torch.zeros((2 * f.numel(), 3), dtype=torch.int32,
                                 device=DEVICE)
    elif kind == "cc_csr":
        n = case["axis"]
        s["row_ptr"], s["col"], perm = _mesh_csr(n, seed)
        f = _mesh_field(n, case["bumps"], seed, perm)
        s["mask"] = (_make_mask(f, case["quantile"])
                     if case["quantile"] > 0 else None)
    elif kind == "segment_csr":
        n = case["axis"]
        s["row_ptr"], s["col"], perm = _mesh_csr(n, seed)
        s["field"] = _mesh_field(n, case["bumps"], seed, perm)
    elif kind == "tets":
        s["tets"] = _mesh_tets(case["axis"], seed)
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "segment":
        if case["check"]:
            return msc.segment(s["field"], want=s["want"])
        msc.segment_into(s["field"], *s["out"], check=False)
        return s["bufs"]
    if kind == "batch":
        msc.segment_batched_into(s["fields"], s["outs"], check=False)
        return s["bufs"]
    if kind == "graph":
        s["graph"].launch()
        return s["bufs"]
    if kind == "cc":
        msc.cc_label_grid_into(s["mask"], s["labels"])
        return s["labels"]
    if kind == "cc_csr":
        return msc.cc_label_csr(s["row_ptr"], s["col"], s["mask"])
    if kind == "segment_csr":
        return msc.segment_csr(s["row_ptr"], s["col"], s["field"],
                               want=s["want"])
    if kind == "tets":
        return msc.csr_from_tets(case["axis"] ** 3, s["tets"])
    code = msc.critical_points(s["field"])
    count = msc.extremum_graph_into(s["field"], s["asc"], s["desc"],
                                    s["edges"])
    return code, s["edges"], count


def work(case):
    """Inputs read once and outputs written once; comparisons of ids and
    values are not counted as floating-point operations."""
    kind = case["kind"]
    outs = len(case["want"].split(",")) if "want" in case else 0
    if kind in ("segment", "cc", "topology"):
        n = case["x"] * case["y"] * case["z"]
        # field and labels; mask and labels; field twice (two calls) and code
        per = {"segment": 4 + 4 * outs, "cc": 1 + 8, "topology": 8 + 1}[kind]
        return dict(bytes=per * n, flops=0)
    if kind in ("batch", "graph"):
        n = sum(d[0] * d[1] * d[2] for d, _ in _specs(case))
        return dict(bytes=(4 + 4 * outs) * n, flops=0)
    m = case["axis"]
    n = m ** 3
    entries = 2 * sum((m - a) * (m - b) * (m - c) for a, b, c in _EDGES)
    graph = 8 * (n + 1) + 4 * entries
    if kind == "cc_csr":
        return dict(bytes=graph + 9 * n, flops=0)
    if kind == "segment_csr":
        return dict(bytes=graph + (4 + 4 * outs) * n, flops=0)
    return dict(bytes=16 * 6 * (m - 1) ** 3 + graph, flops=0)
