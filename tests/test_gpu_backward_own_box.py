"""The backward through the sites' own box at the sizes where the sums over its
faces change shape: one block up to 4096 slots, two kernels above, several
cells a slot beyond 65536 sites.

With the same box given and not given the gradients differ by the sums of
dL/db over each face alone, at the lowest-index site on that face.  The
reference of those sums is FP64: a facet of area A and centroid Y adds
A (g_vol + g_cen . (Y - c) / V), a vertex of the planes M x = b the face's
component of M^-T g_vert.  Areas and centroids come from vertices rounded to
FP32, 6e-8 against edges of 0.02, so 5e-5 of the sum of the absolute terms is
above their rounding and below the share of one cell of a face (3e-4 and
more)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _face_sums(d, xyz, g_vol, g_cen, g_vert):
    """(sums [6], sums of absolute terms [6]) of dL/db over the box faces."""
    import torch
    n = len(xyz)
    cells = torch.arange(n, device="cuda")
    facet_cell = torch.repeat_interleave(cells, torch.diff(d.facet_off))
    box = (d.facet_nbr < 0).nonzero()[:, 0]
    cell, face = facet_cell[box], (-d.facet_nbr[box].long() - 1)
    p, v = xyz.double(), d.vert.double()
    start, size = d.fv_off[box], d.fv_off[box + 1] - d.fv_off[box]
    area = torch.zeros(len(box), dtype=torch.float64, device="cuda")
    moment = torch.zeros((len(box), 3), dtype=torch.float64, device="cuda")
    a = v[d.fv[start].long()]
    for t in range(1, int(size.max()) - 1):
        on = t + 1 < size
        b, c = v[d.fv[(start + t) * on].long()], v[d.fv[(start + t + 1) * on].long()]
        tri = 0.5 * torch.linalg.cross(b - a, c - a).norm(dim=1) * on
        area += tri
        moment += tri[:, None] * (a + b + c) / 3.0
    c, vol, gc = d.centroid.double()[cell], d.vol.double()[cell], g_cen.double()[cell]
    term = area * g_vol.double()[cell] + (gc * (moment - area[:, None] * c)).sum(1) / vol
    terms, faces = [term], [face]
    if g_vert is not None:
        vert_cell = torch.repeat_interleave(cells, torch.diff(d.vert_off))
        rows = (d.vert_planes < 0).any(1).nonzero()[:, 0]
        code, own = d.vert_planes[rows].long(), p[vert_cell[rows]]
        eye = torch.eye(3, dtype=torch.float64, device="cuda")
        out = torch.stack([-eye[0], eye[0], -eye[1], eye[1], -eye[2], eye[2]])
        normal = torch.where((code >= 0)[..., None], p[code.clamp(min=0)] - own[:, None], out[(-code - 1).clamp(min=0)])
        lam = torch.linalg.solve(normal.transpose(1, 2), g_vert.double()[rows])
        for k in range(3):
            on = code[:, k] < 0
            terms.append(lam[on, k])
            faces.append(-code[on, k] - 1)
    term, face = torch.cat(terms), torch.cat(faces)
    zero = torch.zeros(6, dtype=torch.float64, device="cuda")
    return zero.index_add(0, face, term), zero.index_add(0, face, term.abs())


@pytest.mark.parametrize("n,vert", [(4095, True), (4096, False), (4097, True), (65_536, False), (65_537, True),
                                    (100_000, False), (150_001, True)])
def test_face_sums(n, vert):
    import torch
    import paper_2605_06408_amd as vd
    gen = torch.Generator().manual_seed(n)
    xyz = torch.rand((n, 3), generator=gen)
    # a face that several sites stand on: its gradient goes to the first of them
    top = torch.randint(0, n, (3,), generator=gen)
    xyz[top, 2] = xyz[:, 2].max()
    x = xyz.cuda()
    lo, hi = xyz.amin(0), xyz.amax(0)
    ctx = vd.Context(0)

    def gradients(box, noalloc):
        d = ctx.build(x, None, box)
        g_vol = torch.randn(n, generator=torch.Generator().manual_seed(1)).cuda()
        g_cen = torch.randn((n, 3), generator=torch.Generator().manual_seed(2)).cuda()
        g_vert = None
        if vert:
            g_vert = torch.stack([torch.cos(3 * d.vert[:, 0]), torch.sin(2 * d.vert[:, 1]), d.vert[:, 0]], 1).contiguous()
        g, _ = ctx.backward(g_vol, g_cen, g_vert)
        if noalloc:
            assert torch.equal(g, ctx.backward(g_vol, g_cen, g_vert, noalloc=True)[0])
        return d, g.double(), (g_vol, g_cen, g_vert)

    d, given, up = gradients(lo.tolist() + hi.tolist(), False)
    own_d, own, _ = gradients(None, n <= 100_000)
    for k in vd.OUTPUT_FIELDS:
        assert torch.equal(getattr(d, k), getattr(own_d, k)), k
    sums, sizes = _face_sums(d, x, *up)
    expect = given.clone()
    tol = torch.full_like(expect, 1e-12)
    for f in range(6):
        axis, side = f >> 1, f & 1
        site = int((xyz[:, axis] == (hi if side else lo)[axis]).nonzero()[0])
        expect[site, axis] += sums[f] if side else -sums[f]
        tol[site, axis] += 5e-5 * float(sizes[f])
    assert bool(((own - expect).abs() <= tol + 2.0 ** -22 * expect.abs()).all())
    # moving every site and the box with them changes nothing but g_cen . c
    rest = own.sum(0) - up[1].double().sum(0)
    if vert:
        rest -= up[2].double().sum(0)
    assert float(rest.abs().max()) <= 1e-6 * float(own.abs().sum())
