"""A candidate of a leaf that meets no vertex of the cell may meet a later one:
a vertex made by a clip can come out, by its rounding, in doubt of a plane
that no vertex was in doubt of before.  In these two cells of more than 64
vertices some sign is in doubt for such vertices only, so the cell has its
FP64 flag exactly if a plane is still tried after cuts that leave every
vertex clear of it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed", [2130, 2731])
def test_candidates_stay(seed):
    import torch
    import paper_2605_06408_amd as vd
    rng = np.random.default_rng(seed)
    n = int(rng.integers(80, 700))
    u = rng.normal(size=(n, 3))
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    if seed == 2130:
        u = np.round(u * 64) / 64
    else:
        u[:, 2] *= 0.3
    xyz = np.concatenate([np.zeros((1, 3)), 0.3 * u]).astype(np.float32)
    d = vd.Context(0).build(torch.from_numpy(xyz).cuda(), None, [-0.5] * 3 + [0.5] * 3, precision=2)
    assert int(d.flags[0]) == vd.FLAG_LARGE | vd.FLAG_FP64
