"""Groups where their kernels change (one workgroup up to 1024 particles, tiles of
16384 and 4096 beyond) and when the calls on one context alternate: first member
and count exactly the oracle's, boxes to the bit (minima and maxima)."""
import numpy as np
import pytest

import oracle
from gpu_helpers import to_dev
from paper_0909_0541_amd import inputs

pytestmark = pytest.mark.gpu


def test_groups_match_oracle(gpu):
    c = gpu.Context()
    for n in (1, 2, 17, 1023, 1024, 1025, 2048, 16383, 16384, 16385, 70000, 20000, 3):
        for dup in (False, True):
            pos = inputs.clustered(n, 3, n_halos=max(1, n // 2048))[0]
            if dup:  # a bucket larger than any group
                pos[: n // 3] = pos[0]
            mass = np.full(n, 1.0 / n)
            t = oracle.Tree(pos, mass)
            c.build_tree(to_dev(pos), to_dev(mass))
            for n_crit in (256, 1, 17, 64):
                assert c.make_groups(n_crit) == t.groups(n_crit)
                ints, box, _, _ = (None if x is None else x.cpu().numpy() for x in c.export_groups())
                first, count, lo, hi = t.group_info()
                order = np.argsort(first, kind="stable")
                assert np.array_equal(ints[:, 0], first[order]) and np.array_equal(ints[:, 1], count[order])
                assert np.array_equal(box[:, :3], lo[order]) and np.array_equal(box[:, 3:], hi[order])


def test_groups_of_many_systems(gpu):
    """More systems than a workgroup has threads, most of them empty or tiny."""
    rng = np.random.default_rng(2)
    sizes = rng.choice([0, 0, 0, 1, 2, 5], 3000)
    sizes[1500] = 300
    off = np.concatenate([[0], np.cumsum(sizes)])
    n = int(off[-1])
    pos, mass = rng.uniform(-1.0, 1.0, (n, 3)), np.full(n, 1.0)
    c = gpu.Context()
    c.build_batch(off, to_dev(pos), to_dev(mass))
    g = c.make_groups(16)
    ints = c.export_groups()[0].cpu().numpy()
    assert np.array_equal(ints[:, 0], np.concatenate([[0], np.cumsum(ints[:, 1])[:-1]])) and ints[:, 1].sum() == n
    assert ints[:, 1].max() <= 16 and g == ints.shape[0]
    small = np.flatnonzero((sizes > 0) & (sizes <= 16))
    assert all(int((ints[:, 2] == s).sum()) == 1 for s in small[::50])
