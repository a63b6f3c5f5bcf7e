"""The hierarchy and the scans at the sizes where their kernels change shape:
one tile and the next (scans of 2048, one-block sort up to 4096, tiles of 1024,
2048 and 4096 keys), levels of block boxes (128 blocks of 64, of 64^2), many
equal codes.  Sorting and minima are exact, so everything is compared exactly."""
import numpy as np
import pytest

from tests.test_gpu_lbvh import _build, _walk

pytestmark = pytest.mark.gpu


def _sites(n, equal, seed):
    rng = np.random.default_rng(seed)
    xyz = rng.random((n, 3)).astype(np.float32)
    if equal:  # coarse positions: runs of equal codes, coincident sites among them
        xyz = (np.floor(xyz * 16) / 16 + 1 / 32).astype(np.float32)
    return xyz, rng.normal(0.0, 1e-4, n).astype(np.float32)


@pytest.mark.parametrize("n,equal", [(33, False), (2049, True), (4095, False), (4096, True), (4097, False),
                                     (8193, True), (262_144, False), (262_145, True), (4_194_305, False)])
def test_sort(n, equal):
    import torch
    xyz, w = _sites(n, equal, n)
    b = _build(xyz, w, [0, 0, 0, 1, 1, 1], 32)
    vals, idx = torch.sort(torch.from_numpy(b["morton"]), stable=True)
    assert np.array_equal(b["sorted_keys"], vals.numpy())
    assert np.array_equal(b["order"].astype(np.int64), idx.numpy())


@pytest.mark.parametrize("n,leaf_size", [(33, 32), (129, 1), (4097, 32), (8192 + 64, 64), (8192 + 129, 5), (530_003, 32)])
def test_node_boxes(n, leaf_size):
    xyz, w = _sites(n, False, n)
    b = _build(xyz, w, [0, 0, 0, 1, 1, 1], leaf_size)
    visits, leaves, records, rng = _walk(b, n)
    assert np.all(visits[visits > 0] == 1) and rng[0] == (0, n - 1)
    assert sum(l - f + 1 for f, l in leaves) == n and max(l - f + 1 for f, l in leaves) <= leaf_size
    order = b["order"].astype(np.int64)
    sp, sw = xyz[order], w[order]
    fl = b["nodes"].view(np.float32)
    for node, s, f, l in records:
        assert np.array_equal(fl[node, s, 0:3], sp[f:l + 1].min(0)), (node, s)
        assert np.array_equal(fl[node, s, 4:7], sp[f:l + 1].max(0)), (node, s)
        assert fl[node, s, 3] == sw[f:l + 1].max(), (node, s)


@pytest.mark.parametrize("n", [1, 2047, 2048, 2049, 6145])
@pytest.mark.parametrize("own_box", [False, True])
def test_offsets(n, own_box):
    """Offsets are the running sums of the rows' lengths, totals the sizes."""
    import torch
    import paper_2605_06408_amd as vd
    if own_box and n < 4:
        pytest.skip("a flat set has no box of its own")
    xyz, w = _sites(n, False, 7)
    ctx = vd.Context(0)
    x = torch.from_numpy(xyz).cuda()
    d = ctx.build(x, None, None if own_box else [0, 0, 0, 1, 1, 1])
    fv_off, fv = d.fv_off.cpu().numpy(), d.fv.cpu().numpy()
    voff, foff, noff = (getattr(d, k).cpu().numpy() for k in ("vert_off", "facet_off", "nbr_off"))
    for off, total in ((voff, d.sizes["n_vert"]), (foff, d.sizes["n_facet"]), (noff, d.sizes["n_nbr"])):
        assert off[0] == 0 and off[-1] == total and np.all(np.diff(off) >= 0)
    assert fv_off[0] == 0 and fv_off[-1] == len(fv) == 3 * d.sizes["n_vert"]
    # every cell is a simple polytope: F facets, 2 F - 4 vertices, its rings over its own vertices
    assert np.array_equal(np.diff(voff), 2 * np.diff(foff) - 4)
    cell_of_entry = np.repeat(np.arange(n), 3 * np.diff(voff))
    assert np.all((fv >= voff[cell_of_entry]) & (fv < voff[cell_of_entry + 1]))
    site_facets = np.add.reduceat((d.facet_nbr.cpu().numpy() >= 0).astype(np.int64), foff[:-1])
    assert np.array_equal(site_facets, np.diff(noff))
    lo, hi = (xyz.min(0), xyz.max(0)) if own_box else (np.zeros(3), np.ones(3))
    assert abs(d.vol.double().sum().item() / float(np.prod((hi - lo).astype(np.float64))) - 1.0) <= 1e-6
