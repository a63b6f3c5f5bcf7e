"""The 64-vertex pass written for the default options against the general one.

A build with work counters runs the general kernels throughout, so the same
input built with and without counters has to give the same diagram to the
last integer; floating outputs come from FP64 sums in another order and are
held to one unit in the last place of FP32 (2^-23 relative to the largest
coordinate, the centroid of a thin cell to 1e-6 of the box).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _input(kind, n, seed):
    from paper_2605_06408_amd import workloads as wl
    if kind == "lattice":  # exact ties
        k = round(n ** (1.0 / 3.0))
        g = (np.arange(k) + 0.5) / 16.0
        xyz = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3).astype(np.float32)
        return xyz, None, np.array([0, 0, 0] + [k / 16.0] * 3)
    if kind == "coincident":
        xyz, w, box = wl.uniform(n, seed)
        xyz[n // 2:] = xyz[:n - n // 2]
        return xyz, w, box
    if kind == "star":  # one site in the middle of a sphere of others: more than 64 vertices
        d = np.random.default_rng(seed).normal(size=(n, 3))
        xyz = (0.5 + 0.3 * d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
        xyz[0] = 0.5
        return xyz, None, np.array([0.0, 0, 0, 1, 1, 1])
    return {"uniform": wl.uniform, "power": wl.power_uniform, "clustered": wl.clustered,
            "surface": wl.surface}[kind](n, seed)


CASES = ([("uniform", n, 32) for n in (1, 2, 31, 32, 33, 63, 64, 65, 4097)] +
         [("uniform", 64, 64), ("uniform", 300, 1), ("uniform", 20_011, 32), ("power", 20_000, 32), ("clustered", 30_000, 32),
          ("surface", 30_000, 32), ("lattice", 13 ** 3, 32), ("coincident", 2001, 32), ("star", 60, 64),
          ("star", 500, 32)])


@pytest.mark.parametrize("kind,n,leaf", CASES)
def test_equals_the_general_pass(kind, n, leaf):
    import torch
    import paper_2605_06408_amd as vd
    xyz, w, box = _input(kind, n, 5)
    x = torch.from_numpy(np.ascontiguousarray(xyz)).cuda()
    ww = None if w is None else torch.from_numpy(w).cuda()
    bbox = [float(v) for v in box]
    ctx = vd.Context(0)
    general = ctx.build(x, ww, bbox, leaf_size=leaf, counters=True)
    d = ctx.build(x, ww, bbox, leaf_size=leaf)
    for k in ("nbr_off", "nbr", "facet_off", "facet_nbr", "fv_off", "fv", "vert_off", "vert_planes", "flags"):
        assert torch.equal(getattr(d, k), getattr(general, k)), k
    assert d.sizes == general.sizes
    size = float(np.abs(box).max())
    assert float((d.vert - general.vert).abs().max() if len(d.vert) else 0.0) <= 2.0 ** -23 * size
    assert float((d.vol - general.vol).abs().max()) <= 2.0 ** -23 * float(general.vol.max())
    assert float((d.centroid - general.centroid).abs().max()) <= 1e-6 * size
    if kind == "star":
        assert d.sizes["n_large"] >= 1
    if kind == "clustered":
        assert d.sizes["n_fp64"] > 0  # cells of the retry list (tight clusters: inconsistent FP32 signs)


def test_path_of_more_than_64_siblings():
    """A chain of 63 sites, one for each bit of the Morton code, over a group
    of sites of one code: the tree is deeper than the lanes of a wave.  Certified
    cells have the oracle's neighbours (those of the chain see the group as one
    point and are beyond FP32)."""
    import torch
    import oracle
    import paper_2605_06408_amd as vd
    rng = np.random.default_rng(3)
    chain = np.zeros((63, 3))
    for b in range(63):
        chain[b, b % 3] = 1.25 * 2.0 ** (20 - b // 3)
    group = rng.random((200, 3)) * 0.5
    xyz = np.concatenate([chain, group]).astype(np.float32)
    box = np.array([0.0, 0, 0] + [2.0 ** 22] * 3)
    ctx = vd.Context(0)
    d = ctx.build(torch.from_numpy(xyz).cuda(), None, [float(v) for v in box], leaf_size=2)
    bvh = ctx.inspect_bvh()
    deepest, todo = 0, [(bvh["root"], 1)]
    while todo:
        node, depth = todo.pop()
        deepest = max(deepest, depth)
        refs = [int(bvh["nodes"][node, s, 7]) & 0xFFFFFFFF for s in range(2)]
        todo += [(r, depth + 1) for r in refs if not r & 0x80000000]
    assert deepest > 64
    ref = oracle.cells(xyz, None, box)
    off, nbr = d.nbr_off.cpu().numpy(), d.nbr.cpu().numpy()
    cert = np.nonzero(ref["margin"] >= 1e-5)[0]
    assert len(cert) >= 150
    for i in cert:
        assert nbr[off[i]:off[i + 1]].tolist() == ref["nbr"][ref["nbr_off"][i]:ref["nbr_off"][i + 1]].tolist(), i
