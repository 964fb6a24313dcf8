"""Second moments where their passes change: subtrees of 256 particles, pieces of
2560 above them, 220 cells above those at once, and beyond 524288 particles
monopole subtrees (512, 8192, 352) with the second moments level by level.
Node records bit for bit the oracle's; second moments to 1e-12 of the larger of
their trace and the cell's mass times its size squared (the roundings of the
centres of mass and of the sums over at most 22 levels, some 100 units of
1.1e-16)."""
import numpy as np
import pytest

import oracle
from gpu_helpers import to_dev
from paper_0909_0541_amd import inputs

pytestmark = pytest.mark.gpu


def _inputs(kind, n):
    rng = np.random.default_rng(n)
    if kind == "clustered":
        return inputs.clustered(n, 3, n_halos=max(1, n // 2048))[0]
    pos = rng.uniform(0.0, 1.0, (n, 3))
    if kind == "buckets":  # a few points that hold many particles, and loose ones
        big = rng.random(n) < 0.7
        pos[big] = rng.uniform(0.0, 1.0, (5, 3))[rng.choice(5, big.sum(), p=[0.5, 0.3, 0.1, 0.06, 0.04])]
        return pos
    # ever closer to a corner: cells one inside the other, each with some particles of its own
    return pos * 2.0 ** -rng.integers(0, 20, (n, 1)).astype(float)


def _check(c, t, n):
    """Every cell's and bucket's record and moments."""
    ints, reals = (x.cpu().numpy() for x in c.export_nodes())
    mom = c.export_moments().cpu().numpy()
    nd, S = t.nodes(), t.second_moments()
    mine = np.flatnonzero((ints[:, 1] == oracle.KIND_CELL) | (ints[:, 1] == oracle.KIND_BUCKET))
    ref = np.flatnonzero(((nd["kind"] == oracle.KIND_CELL) & (nd["nchild"] > 1)) | (nd["kind"] == oracle.KIND_BUCKET))
    a = ref[np.lexsort((nd["count"][ref], nd["first"][ref]))]
    b = mine[np.lexsort((ints[mine, 3], ints[mine, 2]))]
    assert np.array_equal(nd["first"][a], ints[b, 2]) and np.array_equal(nd["count"][a], ints[b, 3]), n
    assert np.array_equal(nd["mass"][a], reals[b, 0]) and np.array_equal(nd["com"][a], reals[b, 1:4]), n
    cell = nd["kind"][a] == oracle.KIND_CELL
    assert np.array_equal(nd["s"][a][cell], reals[b, 5][cell]), n
    l = np.where(np.isfinite(reals[b, 4]), reals[b, 4], t.info()["side"] * 2.0**-21)
    scale = np.maximum(S[a, :3].sum(1), np.maximum(reals[b, 0] * l * l, 1e-300))
    assert np.all(np.abs(mom[b] - S[a]).max(1) <= 1e-12 * scale), n


@pytest.mark.parametrize("kind", ["clustered", "buckets", "chain"])
@pytest.mark.parametrize("n", [2, 255, 256, 257, 511, 512, 513, 2559, 2560, 2561, 16384, 16385, 100001, 524288, 524289])
def test_edges(gpu, kind, n):
    pos, mass = _inputs(kind, n), np.random.default_rng(1).uniform(0.5, 1.5, n)
    mass[:: max(2, n // 7)] = 0.0
    t = oracle.Tree(pos, mass)
    c = gpu.Context(quadrupole=True)
    c.build_tree(to_dev(pos), to_dev(mass))
    _check(c, t, n)


@pytest.mark.parametrize("pad", [0, 400000])
def test_cells_above_the_pieces(gpu, pad):
    """Batches with just as many cells of more than 2560 particles as are taken at
    once, and with more; padded by another system, of more than 524288 in all
    (the monopole passes' own limits)."""
    one = _inputs("chain", 8000)
    mass = np.random.default_rng(1).uniform(0.5, 1.5, 8000)
    t = oracle.Tree(one, mass)
    nd = t.nodes()
    high = int(((nd["nchild"] > 1) & (nd["count"] > 2560)).sum())
    assert high >= 10
    f = gpu.Context(quadrupole=True)
    f.build_tree(to_dev(one), to_dev(mass))
    _check(f, t, 8000)
    want, want_mom = f.export_nodes(), f.export_moments()
    for k in (220 // high, 220 // high + 1, 40):
        sizes = [8000] * k + ([pad] if pad else [])
        off = np.concatenate([[0], np.cumsum(sizes)])
        pos, m = np.tile(one, (k, 1)), np.tile(mass, k)
        if pad:
            pos, m = np.concatenate([pos, _inputs("clustered", pad)]), np.concatenate([m, np.full(pad, 1.0)])
        assert not pad or off[-1] > 524288 or k < 16
        b = gpu.Context(quadrupole=True)
        b.build_batch(off, to_dev(pos), to_dev(m))
        (ints, reals), mom = b.export_nodes(), b.export_moments()
        for s in (0, k // 2, k - 1):
            # the system's slots by particle range: as in the tree of its own
            i = ((ints[:, 2] >= off[s]) & (ints[:, 2] + ints[:, 3] <= off[s + 1])).nonzero()[:, 0]
            key = (ints[i, 2] - int(off[s])).long() * 8001 + ints[i, 3]
            i = i[key.argsort(stable=True)]
            w = ((want[0][:, 2]).long() * 8001 + want[0][:, 3]).argsort(stable=True)
            assert (reals[i] == want[1][w]).all() and (mom[i] == want_mom[w]).all(), (k, s)
