"""Systems of up to 6500 particles have no outliers, whatever else is in their
batch; against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from gpu_helpers import check_forces, to_dev
from paper_0909_0541_amd import inputs

pytestmark = pytest.mark.gpu


def _spread(n, seed):
    """A ball and seven lone particles in the other octants of its cube: one
    group whose list is every particle."""
    pos = inputs.uniform_sphere(n - 7, seed)[0]
    corners = np.array([[x, y, z] for x in (0.0, 1.0) for y in (0.0, 1.0) for z in (0.0, 1.0)])[:7]
    pos = np.concatenate([corners, 0.7 + 0.1 * pos])
    pos[-1] = 1.0
    return pos


@pytest.mark.parametrize("quad", [False, True])
@pytest.mark.parametrize("sizes,outliers", [([6500], 0), ([6501], 1), ([6500] * 4, 0), ([6501] * 3, 3),
                                            ([6500, 20, 6501, 6500, 9000], 2)])
def test_sizes(gpu, sizes, outliers, quad):
    off = np.concatenate([[0], np.cumsum(sizes)])
    parts = [_spread(n, 3 + k) for k, n in enumerate(sizes)]
    c = gpu.Context(quadrupole=quad)
    c.build_batch(off, to_dev(np.concatenate(parts)), to_dev(np.concatenate([np.full(n, 1.0 / n) for n in sizes])))
    c.make_groups(64)
    a, p = (v.cpu().numpy().astype(np.float64) for v in c.compute_forces_batch([1e-2] * len(sizes), [0.8] * len(sizes)))
    st = c.get_stats()
    assert st.error_flags == 0 and st.n_split_groups == outliers
    inter = 0
    for k, n in enumerate(sizes):
        t = oracle.Tree(parts[k], np.full(n, 1.0 / n))
        t.groups(64)
        ref = t.forces(1e-2, 0.8, quadrupole=quad)
        inter += int(ref["interactions"])
        check_forces(a[off[k]:off[k + 1]], p[off[k]:off[k + 1]], ref)
    assert st.interactions == inter
