"""The 64-vertex pass with checked signs (mixed precision, from 65536 sites)
against the general one, which builds with work counters run throughout: the
same diagram and flags to the last integer (the cells with a doubtful sign
are built by the general pass in both), floats to one unit in the last place
of FP32 (their FP64 sums run in another order; centroids of thin cells to
1e-6 of the box)."""
import numpy as np
import pytest

from .test_gpu_clip64 import _input

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n", [("uniform", 65_535), ("uniform", 65_536), ("power", 70_001), ("clustered", 80_000),
                                    ("surface", 90_001), ("lattice", 41 ** 3), ("coincident", 66_001)])
def test_equals_the_general_pass(kind, n):
    import torch
    import paper_2605_06408_amd as vd
    xyz, w, box = _input(kind, n, 6)
    x = torch.from_numpy(np.ascontiguousarray(xyz)).cuda()
    ww = None if w is None else torch.from_numpy(w).cuda()
    bbox = [float(v) for v in box]
    ctx = vd.Context(0)
    general = ctx.build(x, ww, bbox, precision=2, counters=True)
    d = ctx.build(x, ww, bbox, precision=2)
    for k in ("nbr_off", "nbr", "facet_off", "facet_nbr", "fv_off", "fv", "vert_off", "vert_planes", "flags"):
        assert torch.equal(getattr(d, k), getattr(general, k)), k
    assert d.sizes == general.sizes and d.sizes["n_fp64"] > 0
    size = float(np.abs(box).max())
    assert float((d.vert - general.vert).abs().max()) <= 2.0 ** -23 * size
    assert float((d.vol - general.vol).abs().max()) <= 2.0 ** -23 * float(general.vol.max())
    assert float((d.centroid - general.centroid).abs().max()) <= 1e-6 * size
