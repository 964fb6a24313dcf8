"""Key order at the edges of the sorts: counting in one launch (up to 16384
particles, own tiles of 32 up to 8192 and of 64 beyond), key passes with tiles
of 1024, 2048 and 4096 keys.  Keys and permutation bit for bit the oracle's, so
equal keys in input order; bad input is still reported."""
import numpy as np
import pytest

import oracle
from gpu_helpers import to_dev
from paper_0909_0541_amd import inputs

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 31, 32, 33, 63, 64, 65, 1023, 1025, 8191, 8192, 8193, 16384, 16385, 262144, 262145, 700000, 700001]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("kind", ["clustered", "repeated"])
def test_key_order(gpu, n, kind):
    if kind == "clustered":
        pos = inputs.clustered(n, 7, n_halos=max(1, n // 4096))[0]
    else:  # a few hundred distinct points, in mixed order
        rng = np.random.default_rng(n)
        pos = rng.uniform(-1.0, 1.0, (300, 3))[rng.integers(0, 300, n)]
    mass = np.full(n, 1.0 / n)
    for curve in (0, 1) if n <= 20000 else (0,):
        c = gpu.Context(curve=curve)
        c.build_tree(to_dev(pos), to_dev(mass))
        keys, perm = c.export_sorted()
        keys_o, perm_o = oracle.Tree(pos, mass, curve=curve).sorted()
        assert np.array_equal(keys.cpu().numpy().view(np.uint64), keys_o)
        assert np.array_equal(perm.cpu().numpy().astype(np.int64), perm_o)


@pytest.mark.parametrize("n", [1, 500, 9000, 20000])
def test_bad_input_is_reported(gpu, n):
    bh = gpu
    pos, mass = inputs.uniform_cube(n, 1)[:2]
    c = bh.Context()
    for what in ("nan", "inf", "mass", "nan mass"):
        p, m = pos.copy(), mass.copy()
        if what == "nan":
            p[n - 1, 2] = np.nan
        elif what == "inf":
            p[n // 2, 0] = -np.inf
        else:
            m[n - 1] = -1.0 if what == "mass" else np.nan
        c.build_tree(to_dev(p), to_dev(m))
        with pytest.raises(bh.BHError) as e:
            c.make_groups(16)
        assert e.value.status == -1
    c.build_tree(to_dev(pos), to_dev(mass))
    assert c.make_groups(16) > 0
