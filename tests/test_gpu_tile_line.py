"""The largest monopole tree whose lists are summed by tiles, and one particle
more, against a wave per group (list tile asked for by option): by tiles the same
FP32 chains, added in FP64 in another order, so at most one rounding to FP32
apart (2^-23 of a result, and of the self potential that is taken out); beyond
the line the same kernels, so the same bits.  Members of the few outlier groups
are left out, which are walked apart from another length on."""
import numpy as np
import pytest
import torch

from gpu_helpers import to_dev
from paper_0909_0541_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [400000, 400001])
def test_line(gpu, n):
    pos, mass = inputs.clustered(n, 3, n_halos=200)[:2]
    x, m = to_dev(pos), to_dev(mass)
    eps, res = 1e-3, []
    for opts in ({}, {"list_tile": 1024}):
        c = gpu.Context(**opts)
        c.build_tree(x, m)
        c.make_groups(256)
        a, p = c.compute_forces(eps, 0.6)
        st = c.get_stats()
        assert st.error_flags == 0 and st.n_split_groups <= 4
        res.append((a.double(), p.double(), st))
    (a, p, s), (b, q, r) = res
    assert s.interactions == r.interactions and s.list_entries == r.list_entries and s.max_list == r.max_list
    if n > 400000:
        assert torch.equal(a, b) and torch.equal(p, q)
        return
    ulp = 2.0**-23
    same = ((a - b).abs() <= ulp * b.abs() + 1e-13 * b.abs().max()).all(1)
    same &= (p - q).abs() <= ulp * (q.abs() + 1e-6 * m / eps) + 1e-13 * q.abs().max()
    assert int((~same).sum()) <= 256 * max(s.n_split_groups, r.n_split_groups)
