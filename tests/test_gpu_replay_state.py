"""Replays of a captured step and eager calls on one context, in any order: each
gives the bits that a context of its own gives."""
import numpy as np
import pytest
import torch

from gpu_helpers import to_dev
from paper_0909_0541_amd import inputs

pytestmark = pytest.mark.gpu

EPS = 1e-3


def _case(n, seed):
    pos, mass = inputs.clustered(n, seed, n_halos=max(1, n // 2048))[:2]
    return to_dev(pos), to_dev(mass)


def _fresh(bh, pos, mass, n_crit, theta, **opts):
    return bh.tree_forces(pos, mass, EPS, theta, n_crit, ctx=bh.Context(**opts))


def _nan(n):
    return (torch.full((n, 3), float("nan"), dtype=torch.float32, device="cuda"),
            torch.full((n,), float("nan"), dtype=torch.float32, device="cuda"))


# sums by list tiles; one wave per group (more than 2048 n_crit particles); the
# workgroup walk, with fewer and with more groups than workgroups
@pytest.mark.parametrize("n,n_crit,quad", [(20000, 64, False), (40000, 16, False), (20000, 64, True),
                                           (100003, 64, True)])
def test_forces_after_a_replay(gpu, n, n_crit, quad):
    """Groups are made, then the captured step is replayed, then the forces are
    asked for at another theta."""
    bh = gpu
    pos, mass = _case(n, 7)
    want = _fresh(bh, pos, mass, n_crit, 0.8, quadrupole=quad)
    c = bh.Context(quadrupole=quad)
    c.graph_capture([0, n], pos, mass, n_crit, EPS, 0.6)
    for k in range(2):
        c.build_tree(pos, mass)
        c.make_groups(n_crit)
        c.graph_launch()
        a, p = c.compute_forces(EPS, 0.8, acc=_nan(n)[0], pot=_nan(n)[1])
        c.sync()
        assert torch.equal(a, want[0]) and torch.equal(p, want[1]), k


def test_features_after_a_replay(gpu):
    """The feature probe takes its groups from the same queues."""
    bh = gpu
    n = 20000
    pos, mass = _case(n, 8)
    c = bh.Context()
    c.build_tree(pos, mass)
    groups = c.make_groups(64)
    want = c.group_features(EPS, groups).clone()  # (and its buffers, before the capture)
    c.graph_capture([0, n], pos, mass, 64, EPS, 0.6)
    c.make_groups(64)
    c.graph_launch()
    assert torch.equal(c.group_features(EPS, groups), want)
