"""Slots and moments where the subtrees (512 or 1024 particles), the pieces above them
(8192; 4096 with second moments), the list of cells above those (176 or 352 at
once) and the scan's tiles end; with buckets above and below these sizes, deep
chains, systems of one particle and empty systems.  Node records bit for bit
the oracle's; second moments to 1e-12 of the larger of their trace and the
cell's mass times its size squared (the roundings of the centres of mass and of
the sums over at most 22 levels, some 100 units of 1.1e-16)."""
import numpy as np
import pytest

import oracle
from gpu_helpers import gpu_nodes, oracle_nonchain_nodes, to_dev
from paper_0909_0541_amd import inputs

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 3, 511, 512, 513, 1023, 1024, 1025, 4096, 4097, 8192, 8193, 16384, 16385, 40000, 100001]


def _inputs(kind, n):
    rng = np.random.default_rng(n)
    if kind == "clustered":
        return inputs.clustered(n, 3, n_halos=max(1, n // 2048))[0]
    if kind == "buckets":  # a few points that hold many particles, and loose ones
        pos = rng.uniform(-1.0, 1.0, (n, 3))
        big = rng.random(n) < 0.7
        pos[big] = rng.uniform(-1.0, 1.0, (5, 3))[rng.choice(5, big.sum(), p=[0.5, 0.3, 0.1, 0.06, 0.04])]
        return pos
    # ever closer to one point: a chain of cells, each with some particles of its own
    return rng.uniform(-1.0, 1.0, (n, 3)) * 2.0 ** -rng.integers(0, 20, (n, 1)).astype(float)


@pytest.mark.parametrize("quad", [False, True])
@pytest.mark.parametrize("kind", ["clustered", "buckets", "chain"])
def test_nodes_match_oracle(gpu, kind, quad):
    for n in SIZES + ([2000000] if kind == "clustered" else []):
        pos = _inputs(kind, n)
        mass = np.random.default_rng(1).uniform(0.5, 1.5, n)
        t = oracle.Tree(pos, mass)
        c = gpu.Context(quadrupole=quad)
        c.build_tree(to_dev(pos), to_dev(mass))
        if n > 200000:  # (the records alone, by numbers: dictionaries of them take minutes)
            st, nd = c.get_stats(), t.nodes()
            ints, reals = (x.cpu().numpy() for x in c.export_nodes())
            cells = (nd["kind"] == oracle.KIND_CELL) & (nd["nchild"] > 1)
            mine = ints[:, 1] == oracle.KIND_CELL
            a = np.lexsort((nd["count"][cells], nd["first"][cells]))
            b = np.lexsort((ints[mine, 3], ints[mine, 2]))
            assert np.array_equal(nd["first"][cells][a], ints[mine, 2][b])
            assert np.array_equal(nd["count"][cells][a], ints[mine, 3][b])
            assert np.array_equal(nd["mass"][cells][a], reals[mine, 0][b])
            assert np.array_equal(nd["com"][cells][a], reals[mine, 1:4][b])
            assert np.array_equal(nd["s"][cells][a], reals[mine, 5][b])
            assert st.n_slots == ints.shape[0]
            continue
        got, ints, reals = gpu_nodes(c)
        assert got == oracle_nonchain_nodes(t), (kind, n)
        if quad:
            mom, nd, S = c.export_moments().cpu().numpy(), t.nodes(), t.second_moments()
            cells = np.flatnonzero(nd["kind"] != oracle.KIND_PARTICLE)
            ref = {(int(nd["first"][k]), int(nd["count"][k])): S[k] for k in cells}
            for k in np.flatnonzero((ints[:, 1] != 1) & (ints[:, 1] != 3)):
                want = ref[(int(ints[k, 2]), int(ints[k, 3]))]
                l = reals[k, 4] if np.isfinite(reals[k, 4]) else t.info()["side"] * 2.0**-21
                scale = max(want[:3].sum(), reals[k, 0] * l * l, 1e-300)
                assert np.max(np.abs(mom[k] - want)) <= 1e-12 * scale, (kind, n, k)


@pytest.mark.parametrize("quad", [False, True])
def test_batch_nodes_equal_standalone(gpu, quad):
    sizes = [0, 1, 513, 0, 9000, 512, 1, 2, 20000, 0]
    off = np.concatenate([[0], np.cumsum(sizes)])
    pos = np.concatenate([_inputs("clustered", k) if k else np.zeros((0, 3)) for k in sizes])
    mass = np.random.default_rng(2).uniform(0.5, 1.5, len(pos))
    b = gpu.Context(quadrupole=quad)
    b.build_batch(off, to_dev(pos), to_dev(mass))
    got, _, _ = gpu_nodes(b)
    want = {}
    for s, k in enumerate(sizes):
        if not k:
            continue
        c = gpu.Context(quadrupole=quad)
        c.build_tree(to_dev(pos[off[s]:off[s + 1]].copy()), to_dev(mass[off[s]:off[s + 1]].copy()))
        for (first, count, level), rec in gpu_nodes(c)[0].items():
            want[(first + int(off[s]), count, level)] = rec
    assert got == want
