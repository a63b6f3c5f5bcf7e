"""Coincident sites: of those at one position the heaviest (ties: the lowest
index) has the cell, the others are empty.  Runs of equal codes shorter and
longer than a wave's 64 positions and across their ends, positions that share
a code without being equal, weights with ties.  The winners are exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _context():
    import paper_2605_06408_amd as vd
    return vd.Context(0)


def _cuda(a):
    import torch
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


def _winners(xyz, w):
    _, place = np.unique(xyz, axis=0, return_inverse=True)
    place = place.reshape(-1)
    best = {}
    for i in np.lexsort((np.arange(len(xyz)), -w)):
        best.setdefault(place[i], i)
    return np.array(sorted(best.values()))


@pytest.mark.parametrize("one_code", [False, True])
@pytest.mark.parametrize("weights", ["none", "ties", "all different"])
@pytest.mark.parametrize("copies", [(2, 1, 3), (63, 1, 64, 65, 5), (64, 64, 128), (127, 129, 191, 1, 1), (1000, 3, 20000)])
def test_heaviest_of_a_position(copies, weights, one_code):
    rng = np.random.default_rng(sum(copies))
    box = [0.0, 0, 0, 1, 1, 1]
    places = rng.random((len(copies), 3))
    if one_code:  # all places in one cell of the code's grid of 2^21 (the background is not)
        box = [0.0] * 3 + [2.0 ** 21] * 3
        places *= 0.9
    xyz = np.concatenate([np.repeat(places, copies, 0), rng.random((37, 3)) * box[3]]).astype(np.float32)
    xyz = xyz[rng.permutation(len(xyz))]
    w = np.zeros(len(xyz), np.float32)
    if weights != "none":
        # far below the squared distance of two places: every winner has a cell
        w = (1e-5 * (rng.integers(0, 3, len(w)) if weights == "ties" else rng.random(len(w)))).astype(np.float32)
    d = _context().build(_cuda(xyz), None if weights == "none" else _cuda(w), box, precision=2 if one_code else 1)
    alive = np.nonzero((d.flags.cpu().numpy() & 1) == 0)[0]
    assert np.array_equal(alive, _winners(xyz, w))
    assert d.sizes["n_empty"] == len(xyz) - len(alive)


def test_time_of_long_runs():
    """The hierarchy of 50 places of 8000 sites each: a wave reads its own 64
    positions and the few winners' waves the 125 times 64 of their run, about
    a millisecond if nothing overlapped; that of as many sites without
    coincident ones takes a quarter of one.  Comparing every site with its whole
    run one by one takes 40 times as long as that and more."""
    rng = np.random.default_rng(5)
    ctx = _context()

    def hierarchy(xyz):
        x, best = _cuda(xyz), np.inf
        for _ in range(6):
            ctx.build_sizes(x, None, [0.0, 0, 0, 1, 1, 1], profile=True)
            best = min(best, ctx.timings()["lbvh"])
        return best

    plain = hierarchy(rng.random((400_000, 3)))
    runs = hierarchy(np.repeat(rng.random((50, 3)), 8000, 0)[rng.permutation(400_000)])
    assert runs <= 8.0 * plain, (runs, plain)
