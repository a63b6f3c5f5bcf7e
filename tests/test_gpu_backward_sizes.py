"""The backward at the sizes where its cell passes change shape: cells of up to
32 facets and more (half a wave, one round or two), cells of the 128-vertex
pass (a wave), of the larger ones (a block), and beyond what a block keeps in
LDS (2048 vertices, 1536 with vertex gradients).

One site stands inside a sphere of n others, so its cell has n facets and
2 n - 4 vertices.  Against the gradient oracle (FP64, from the same FP32
inputs) the difference is the rounding of the outputs to FP32 (2^-24) and the
FP64 error of the sums: 1e-6 of the largest component is far above both."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,vert", [(6, False), (31, False), (33, True), (34, False), (36, True), (63, False),
                                    (66, True), (70, False), (300, True), (900, True), (1100, False)])
def test_star(n, vert):
    import torch
    import oracle
    import paper_2605_06408_amd as vd
    from oracle import grad as og
    rng = np.random.default_rng(n)
    d = rng.normal(size=(n, 3))
    xyz = np.concatenate([[[0.5, 0.5, 0.5]], 0.5 + 0.3 * d / np.linalg.norm(d, axis=1, keepdims=True)])
    xyz = xyz.astype(np.float32)
    w = rng.normal(0.0, 1e-4, n + 1).astype(np.float32)
    w[1:] *= 0.01
    box = np.array([0.0, 0, 0, 1, 1, 1])
    ctx = vd.Context(0)
    # doubtful signs in FP64: the combinatorics are then the oracle's
    dg = ctx.build(torch.from_numpy(xyz).cuda(), torch.from_numpy(w).cuda(), [float(v) for v in box], precision=2)
    ref = oracle.cells(xyz, w, box)
    assert np.array_equal(dg.vert_off.cpu().numpy(), ref["vert_off"])
    assert np.array_equal(dg.nbr.cpu().numpy(), ref["nbr"])

    def field(x):  # vertex gradients by position
        return np.stack([np.cos(3 * x[..., 0]), np.sin(2 * x[..., 1]), x[..., 0] * x[..., 2]], -1)

    def cuda(a):
        return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()

    g_vol = rng.normal(size=n + 1).astype(np.float32)
    g_cen = rng.normal(size=(n + 1, 3)).astype(np.float32)
    gx = cuda(field(dg.vert.cpu().numpy().astype(np.float64))) if vert else None
    got_x, got_w = ctx.backward(cuda(g_vol), cuda(g_cen), gx)
    again_x, again_w = ctx.backward(cuda(g_vol), cuda(g_cen), gx, noalloc=True)
    assert torch.equal(got_x, again_x) and torch.equal(got_w, again_w)
    op, ow, _ = og.backward(xyz, w, box, g_vol.astype(np.float64), g_cen.astype(np.float64),
                            (lambda x, codes, i: field(x)) if vert else None)
    px, pw = got_x.cpu().numpy().astype(np.float64), got_w.cpu().numpy().astype(np.float64)
    tol = 1e-6 if not vert else 1e-5  # the field is taken at FP32 positions
    assert np.abs(px - op).max() <= tol * np.abs(op).max()
    assert np.abs(pw - ow).max() <= tol * np.abs(ow).max()
