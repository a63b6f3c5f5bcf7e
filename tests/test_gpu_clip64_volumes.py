"""Volumes and centroids of the 64-vertex pass of vd_clip64.hip, cell by cell,
against the general pass (builds with work counters): both sum FP64 terms of
the same vertices, in another order in FP32 builds.  A cell of size e has
terms of up to e^3, so its volume may differ by their rounding, 64 terms of
2^-53 e^3, and by one unit in the last place of the FP32 output; the centroid by
64 terms of 2^-53 e^4 over four times the volume, and one unit of its own
rounding."""
import numpy as np
import pytest

from .test_gpu_clip64 import _input

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,precision", [("clustered", 30_000, 1), ("clustered", 80_000, 2), ("surface", 30_000, 1),
                                              ("surface", 90_001, 2), ("power", 20_000, 1), ("uniform", 20_011, 1),
                                              ("lattice", 13 ** 3, 1), ("lattice", 41 ** 3, 2)])
def test_cell_by_cell(kind, n, precision):
    import torch
    import paper_2605_06408_amd as vd
    xyz, w, box = _input(kind, n, 5)
    x = torch.from_numpy(np.ascontiguousarray(xyz)).cuda()
    ww = None if w is None else torch.from_numpy(w).cuda()
    ctx = vd.Context(0)
    general = ctx.build(x, ww, [float(v) for v in box], precision=precision, counters=True)
    d = ctx.build(x, ww, [float(v) for v in box], precision=precision)
    assert torch.equal(d.vert_off, general.vert_off)
    count = torch.diff(d.vert_off)
    live = count > 0
    cell = torch.repeat_interleave(torch.arange(len(count), device="cuda"), count)
    lo = torch.full((len(count), 3), float("inf"), device="cuda")
    hi = -lo
    lo = lo.scatter_reduce(0, cell[:, None].expand(-1, 3), d.vert, "amin")
    hi = hi.scatter_reduce(0, cell[:, None].expand(-1, 3), d.vert, "amax")
    size = (hi - lo).double().norm(dim=1)[live]
    a, b = d.vol.double()[live], general.vol.double()[live]
    assert float(b.min()) > 0.0
    assert bool(((a - b).abs() <= 2.0 ** -23 * b + 2.0 ** -47 * size ** 3).all())
    a, c = d.centroid.double()[live], general.centroid.double()[live]
    tol = 2.0 ** -23 * c.abs() + (2.0 ** -47 * size ** 4 / (4.0 * b))[:, None]
    assert bool(((a - c).abs() <= tol).all())
    assert torch.equal(d.centroid[~live], general.centroid[~live]) and not d.vol[~live].any()
