"""Sums by list tiles, taken with few groups (with quadrupoles by a context that
integrates), against the sums of one wave per group (list tile asked for by option) over the
same lists: the FP32 chains are the same and only FP64 partial sums are added in
another order, so a result differs by at most one rounding to FP32 (2^-23 of
it, and of the self potential that is taken out).  Statistics are equal."""
import numpy as np
import pytest
import torch

from gpu_helpers import to_dev
from paper_0909_0541_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("quad", [False, True])
@pytest.mark.parametrize("n,n_crit,theta", [(16, 16, 0.6), (1000, 16, 0.0), (3000, 64, 0.0), (4000, 64, 0.3),
                                            (20000, 100, 0.6), (60001, 256, 0.5), (130000, 64, 0.7)])
def test_tiles_equal_single_waves(gpu, n, n_crit, theta, quad):
    pos = inputs.clustered(n, 3, n_halos=max(1, n // 2048))[0]
    mass = np.random.default_rng(1).uniform(0.5, 1.5, n) / n
    eps = 1e-3
    res = []
    for integrates in (True, False):
        c = gpu.Context(quadrupole=quad) if integrates else gpu.Context(quadrupole=quad, list_tile=1024)
        x, m = to_dev(pos), to_dev(mass)
        if integrates:
            c.kick(torch.zeros_like(x), torch.zeros((n, 3), dtype=torch.float32, device=x.device), 0.0)
        for _ in range(2):  # (the second call's pools hold every list at once)
            c.build_tree(x, m)
            c.make_groups(n_crit)
            acc, pot = c.compute_forces(eps, theta)
        st = c.get_stats()
        assert st.error_flags == 0
        res.append((acc.double(), pot.double(), st))
    (a, p, s), (b, q, r) = res
    outliers = s.n_split_groups + r.n_split_groups
    assert outliers <= 4
    for k in ("interactions", "list_entries", "max_list", "near_entries", "n_groups") + (() if outliers else ("node_visits",)):
        assert getattr(s, k) == getattr(r, k), k
    ulp = 2.0**-23
    self_pot = torch.as_tensor(mass, device=p.device) / eps
    same = ((a - b).abs() <= ulp * b.abs() + 1e-13 * b.abs().max()).all(1)
    same &= (p - q).abs() <= ulp * (q.abs() + 1e-6 * self_pot) + 1e-13 * q.abs().max()
    assert int((~same).sum()) <= outliers * n_crit
    assert float((a - b).norm(dim=1).max()) <= 1e-5 * float(b.norm(dim=1).max())
    assert float((p - q).abs().max()) <= 1e-5 * float(q.abs().max())
