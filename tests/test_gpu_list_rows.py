"""First calls whose pool of list blocks is too small: lists that fit and lists
that do not end in any order.  The walk's rows must stay within the pool (the
call checks the counters it reads back), and the walk after it gives what a
second call gives, and at theta = 0 the direct sums."""
import numpy as np
import pytest
import torch

from gpu_helpers import to_dev
from paper_0909_0541_amd import inputs

pytestmark = pytest.mark.gpu


# small groups: many more blocks needed than there are, a short row for each
@pytest.mark.parametrize("n,n_crit,theta", [(20000, 16, 0.0), (32768, 16, 0.1), (60000, 64, 0.1), (9000, 256, 0.0)])
def test_workgroup_walk(gpu, n, n_crit, theta):
    pos, mass = inputs.clustered(n, 4, n_halos=8)[:2]
    x, m = to_dev(pos), to_dev(mass)
    c = gpu.Context(quadrupole=True)
    c.build_tree(x, m)
    c.make_groups(n_crit)
    a, p = (v.clone() for v in c.compute_forces(1e-3, theta))
    st = c.get_stats()
    assert st.error_flags == 0 and (st.n_walk_attempts > 1) == (n != 9000)
    b, q = c.compute_forces(1e-3, theta)
    assert c.get_stats().n_walk_attempts == 1
    assert torch.equal(a, b) and torch.equal(p, q)
    if theta == 0.0:
        idx = torch.arange(0, n, 37, device="cuda")
        ref, refp = c.direct_sampled(x, m, 1e-3, idx)
        # FP32 sums of n terms, at most 256 at a time before they go to FP64, each
        # off by a few roundings of its own size
        scale = ref.norm(dim=1, keepdim=True) + ref.norm(dim=1).mean()
        assert float(((a[idx].double() - ref).abs() / scale).max()) <= 1e-5
        assert float(((p[idx].double() - refp).abs() / refp.abs()).max()) <= 1e-5


@pytest.mark.parametrize("n,n_crit", [(30000, 16), (40000, 8), (60000, 3)])
def test_outliers(gpu, n, n_crit):
    """Six hundred lone particles around a ball: up to hundreds of groups with
    lists of nearly everything, below and above the sizes summed by tiles."""
    rng = np.random.default_rng(3)
    shell = rng.normal(size=(600, 3))
    shell *= (4.0 + rng.random((600, 1))) / np.linalg.norm(shell, axis=1, keepdims=True)
    pos = np.concatenate([inputs.uniform_sphere(n - 600, 5)[0] * 0.5, shell])
    x, m = to_dev(pos), to_dev(np.full(n, 1.0 / n))
    c = gpu.Context()
    c.build_tree(x, m)
    c.make_groups(n_crit)
    a, p = (v.clone() for v in c.compute_forces(1e-3, 0.3))
    assert c.get_stats().error_flags == 0
    b, q = c.compute_forces(1e-3, 0.3)
    assert c.get_stats().error_flags == 0
    assert torch.equal(a, b) and torch.equal(p, q)
