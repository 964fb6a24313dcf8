"""Per-particle walk where its bundles end (16 particles up to 2^18 of them,
32 beyond), with coincident particles, against the group walk over groups of
one particle: the same terms, so equal statistics and forces within the FP32
force bar (1e-5 of the largest; the longest lists here hold 2e4 terms)."""
import numpy as np
import pytest

from gpu_helpers import to_dev
from paper_0909_0541_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,theta", [
    ("plummer", 1, 0.6), ("plummer", 2, 0.0), ("plummer", 15, 0.3), ("plummer", 16, 0.6), ("plummer", 17, 1.0),
    ("plummer", 1000, 0.0), ("repeated", 5000, 0.5), ("plummer", 20000, 0.8), ("clustered", 262144, 0.7),
    ("clustered", 262145, 0.7), ("repeated", 300001, 0.9)])
def test_bundles_equal_groups_of_one(gpu, kind, n, theta):
    rng = np.random.default_rng(n)
    if kind == "repeated":  # a fifth of the particles at 40 points
        pos = rng.uniform(-1.0, 1.0, (n, 3))
        same = rng.random(n) < 0.2
        pos[same] = rng.uniform(-1.0, 1.0, (40, 3))[rng.integers(0, 40, same.sum())]
    elif kind == "plummer":
        pos = inputs.plummer(n, 3, with_vel=False)[0]
    else:
        pos = inputs.clustered(n, 3, n_halos=n // 2048)[0]
    mass = rng.uniform(0.5, 1.5, n) / n
    c = gpu.Context()
    c.build_tree(to_dev(pos), to_dev(mass))
    a, p = c.compute_forces_particle(1e-2, theta)
    s = c.get_stats()
    c.make_groups(1)
    b, q = c.compute_forces(1e-2, theta)
    r = c.get_stats()
    assert s.error_flags == 0 and r.error_flags == 0
    for k in ("interactions", "list_entries", "max_list"):
        assert getattr(s, k) == getattr(r, k), k
    assert float((a - b).norm(dim=1).max()) <= 1e-5 * float(b.norm(dim=1).max())
    assert float((p - q).abs().max()) <= 1e-5 * float(q.abs().max())
