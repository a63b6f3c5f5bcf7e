"""Mixed precision on sets full of ties, where the 64-vertex pass of
vd_clip64.hip leaves most cells to the general one: which cells it tries
depends on the order in which waves take them, so it must not show.  Against
a build by the general pass alone (work counters) and against itself, every
output to the last bit, floats included (both sum in the same order).

A lattice of 80^3 is 83 cells a wave: the list of a wave is handed on in the
middle of its cells."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _lattice(k, rng):
    g = (np.arange(k) + 0.5) / 64.0
    xyz = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
    return xyz[rng.permutation(len(xyz))], [0.0, 0, 0] + [k / 64.0] * 3


def _input(kind, n, rng):
    from paper_2605_06408_amd import workloads as wl
    if kind == "lattice":
        xyz, box = _lattice(n, rng)
    elif kind == "half":  # the lower half of the lattice replaced by random sites
        xyz, box = _lattice(n, rng)
        low = xyz[:, 0] < 0.5 * box[3]
        xyz[low] = rng.random((int(low.sum()), 3)) * [0.5 * box[3], box[4], box[5]]
    elif kind == "grid":  # random places of a grid, some twice
        xyz, box = (rng.integers(0, 128, (n, 3)) + 0.5) / 128.0, [0.0, 0, 0, 1, 1, 1]
    else:
        xyz, w, box = getattr(wl, kind)(n, 3)
        return xyz, w, [float(v) for v in box]
    return xyz.astype(np.float32), None, box


@pytest.mark.parametrize("kind,n", [("lattice", 41), ("lattice", 64), ("lattice", 80), ("half", 64), ("grid", 200_000),
                                    ("uniform", 200_003), ("surface", 150_001), ("clustered", 100_001),
                                    ("power_uniform", 100_003)])
def test_route_does_not_show(kind, n):
    import torch
    import paper_2605_06408_amd as vd
    xyz, w, box = _input(kind, n, np.random.default_rng(n))
    x = torch.from_numpy(np.ascontiguousarray(xyz)).cuda()
    ww = None if w is None else torch.from_numpy(w).cuda()
    ctx = vd.Context(0)
    general = ctx.build(x, ww, box, precision=2, counters=True)
    if kind == "lattice":
        assert general.sizes["n_fp64"] == n ** 3  # every cell has a tie
        assert int(torch.diff(general.nbr_off).min()) >= 3
    for _ in range(2):
        d = ctx.build(x, ww, box, precision=2)
        assert d.sizes == general.sizes
        for k in vd.OUTPUT_FIELDS:
            a, b = getattr(d, k), getattr(general, k)
            if a.dtype == torch.float32:  # bits, so that a NaN equals itself
                a, b = a.view(torch.int32), b.view(torch.int32)
            assert torch.equal(a, b), k


def test_passes_run_again():
    """More cells beyond 128 vertices than a fresh context has room for (1024):
    the passes run a second time, over the marks and lists of the first.  1600
    sites, each inside a sphere of 70 others, on a lattice of spheres."""
    import torch
    import paper_2605_06408_amd as vd
    rng = np.random.default_rng(8)
    g = np.stack(np.meshgrid(np.arange(16), np.arange(10), np.arange(10), indexing="ij"), -1).reshape(-1, 1, 3) + 0.5
    u = rng.normal(size=(len(g), 70, 3))
    u *= 0.2 / np.linalg.norm(u, axis=2, keepdims=True)
    xyz = np.concatenate([g, g + u], 1).reshape(-1, 3)
    xyz = torch.from_numpy(xyz[rng.permutation(len(xyz))].astype(np.float32)).cuda()
    box = [0.0, 0, 0, 16, 10, 10]
    fresh = vd.Context(0).build(xyz, None, box, precision=2)
    assert int((torch.diff(fresh.vert_off) > 128).sum()) > 1024
    ctx = vd.Context(0)
    general = ctx.build(xyz, None, box, precision=2, counters=True)
    again = ctx.build(xyz, None, box, precision=2)
    for k in vd.OUTPUT_FIELDS:
        assert torch.equal(getattr(fresh, k), getattr(general, k)), k
        assert torch.equal(getattr(again, k), getattr(general, k)), k
