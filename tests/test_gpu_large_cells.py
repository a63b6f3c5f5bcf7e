"""Cells built by several waves together, at the sizes where a wave's slots
pass from one store to another: 128 and 1024 vertices (the ends of passes),
2048 (the slots a group of eight waves keeps in registers), 4096 (slots
counted in one round of a wave), and clips of more new vertices than a wave
has lanes (64) or the lists in LDS have places (1024).

The references are exact counts: a site in the middle of a sphere of n others
has them all as neighbours and 2 n - 4 vertices; a site on the axis of a
ring of n others with one more site above and one below has a prism of n + 2
facets and 2 n vertices.  Volumes are held to 1e-6 of an FP64 evaluation from
the input coordinates (stored as FP32, 6e-8, from FP64 sums; a vertex wrongly
decided by FP32 moves no more than that)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _build(xyz, box, precision):
    import torch
    import paper_2605_06408_amd as vd
    ctx = vd.Context(0)
    d = ctx.build(torch.from_numpy(np.ascontiguousarray(xyz)).cuda(), None, box, precision=precision)
    assert d.sizes["n_failed"] == 0
    return d


def _cell0(d):
    nbr = d.nbr[int(d.nbr_off[0]):int(d.nbr_off[1])].cpu().numpy()
    nf = int(d.facet_off[1] - d.facet_off[0])
    nv = int(d.vert_off[1] - d.vert_off[0])
    fv = d.fv_off[int(d.facet_off[0]):int(d.facet_off[1]) + 1].cpu().numpy()
    return nbr, nf, nv, np.diff(fv), float(d.vol[0])


@pytest.mark.parametrize("n,precision", [(n, 1) for n in (65, 66, 67, 200, 513, 514, 515, 1025, 1027, 2049, 2051, 8000)] +
                         [(700, 2), (2200, 2)])
def test_sphere(n, precision):
    from scipy.spatial import ConvexHull
    u = np.random.default_rng(n).normal(size=(n, 3))
    xyz = np.concatenate([np.zeros((1, 3)), 0.3 * u / np.linalg.norm(u, axis=1, keepdims=True)]).astype(np.float32)
    d = _build(xyz, [-0.5] * 3 + [0.5] * 3, precision)
    assert abs(float(d.vol.double().sum()) - 1.0) < 1e-5
    nbr, nf, nv, sizes, vol = _cell0(d)
    assert nbr.tolist() == list(range(1, n + 1)) and nf == n and nv == 2 * n - 4
    assert sizes.min() >= 3 and sizes.sum() == 3 * nv
    # the cell is the polar of the sites' hull: a vertex for each triangle
    a = xyz[1:].astype(np.float64)
    b = 0.5 * (a * a).sum(1)
    tri = ConvexHull(a).simplices
    v = np.linalg.solve(a[tri], b[tri][..., None])[..., 0]
    assert vol == pytest.approx(ConvexHull(v).volume, rel=1e-6)


@pytest.mark.parametrize("n,precision", [(60, 1), (64, 1), (65, 1), (100, 1), (511, 1), (600, 1), (300, 2), (900, 2), (1500, 2)])
def test_prism(n, precision):
    t = 2.0 * np.pi * (np.arange(n) + 0.2 * np.random.default_rng(n).random(n)) / n
    ring = 0.2 * np.stack([np.cos(t), np.sin(t), np.zeros(n)], 1)
    xyz = np.concatenate([np.zeros((1, 3)), ring, [[0, 0, 0.48], [0, 0, -0.46]]]).astype(np.float32)
    nbr, nf, nv, sizes, vol = _cell0(_build(xyz, [-0.5] * 3 + [0.5] * 3, precision))
    assert nbr.tolist() == list(range(1, n + 3)) and nf == n + 2 and nv == 2 * n
    assert sorted(sizes.tolist()) == [4] * n + [n, n]
    p = xyz[1:n + 1, :2].astype(np.float64)
    q = np.roll(p, -1, 0)
    c = np.linalg.solve(np.stack([p, q], 1), 0.5 * np.stack([(p * p).sum(1), (q * q).sum(1)], 1)[..., None])[..., 0]
    area = 0.5 * abs((c[:, 0] * np.roll(c[:, 1], -1) - c[:, 1] * np.roll(c[:, 0], -1)).sum())
    h = 0.5 * (float(xyz[n + 1, 2]) - float(xyz[n + 2, 2]))
    assert vol == pytest.approx(area * h, rel=1e-6)
