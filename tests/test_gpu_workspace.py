"""Workspaces that follow the tree: rows of list tiles sized for this tree's lists
and grown when they need more, outliers' tables made when there are outliers (or
a captured step may meet them)."""
import numpy as np
import pytest
import torch

from gpu_helpers import to_dev
from paper_0909_0541_amd import inputs

pytestmark = pytest.mark.gpu


def test_small_tree_after_a_large_one(gpu):
    """The list pools of 2 million particles hold some hundred thousand chunks;
    390,000 particles in groups of 256 have about 20,000 tiles, 8 KiB of partial
    sums each."""
    c = gpu.Context()
    x, m = (to_dev(v) for v in inputs.clustered(2000000, 3, n_halos=500)[:2])
    gpu.tree_forces(x, m, 1e-3, 0.35, 256, ctx=c)
    x, m = x[:390000].contiguous(), m[:390000].contiguous()
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    a, p = gpu.tree_forces(x, m, 1e-3, 0.6, 256, ctx=c)
    torch.cuda.synchronize()
    assert free - torch.cuda.mem_get_info()[0] < 400 << 20
    b, q = gpu.tree_forces(x, m, 1e-3, 0.6, 256)
    assert torch.equal(a, b) and torch.equal(p, q)


@pytest.mark.parametrize("n,n_crit", [(3000, 16), (20000, 64), (20000, 256)])
def test_tile_rows_grow(gpu, n, n_crit):
    """Lists by a per-group theta far below the call's: more tiles than expected.
    The walk runs again, and later calls have the room."""
    bh = gpu
    x, m = (to_dev(v) for v in inputs.clustered(n, 5, n_halos=8)[:2])
    want = bh.tree_forces(x, m, 1e-3, 0.125, n_crit)
    tg = torch.full((n,), 0.125, dtype=torch.float32, device="cuda")
    c = bh.Context()
    for k in range(2):
        c.build_tree(x, m)
        c.make_groups(n_crit)
        a, p = c.compute_forces(1e-3, 1.0, theta_group=tg)
        assert torch.equal(a, want[0]) and torch.equal(p, want[1])
        assert (c.get_stats().n_walk_attempts > 1) == (k == 0)
    acc, pot = c.graph_capture([0, n], x, m, n_crit, 1e-3, 1.0, theta_group=tg)
    for _ in range(2):
        acc.zero_()
        c.graph_launch()
        c.sync()
        assert torch.equal(acc, want[0]) and torch.equal(pot, want[1])


@pytest.mark.parametrize("n", [8192, 30000, 450000])
def test_captured_step_meets_outliers(gpu, n):
    """A step captured without outliers has room for some all the same."""
    bh = gpu
    x, m = (to_dev(v) for v in inputs.uniform_sphere(n, 4)[:2])
    pos = to_dev(inputs.plummer(n, 4, with_vel=False)[0])
    want = bh.tree_forces(pos, m, 1e-3, 0.7, 64)
    c = bh.Context(split_visits=-1)
    bh.tree_forces(pos, m, 1e-3, 0.7, 64, ctx=c)  # (its list pools, without outliers)
    c.set_options(split_visits=0)
    acc, pot = c.graph_capture([0, n], x, m, 64, 1e-3, 0.7)
    assert c.get_stats().n_split_groups == 0
    x.copy_(pos)
    for _ in range(2):
        acc.zero_()
        c.graph_launch()
        c.sync()
        assert c.get_stats().n_split_groups > 0
        assert torch.equal(acc, want[0]) and torch.equal(pot, want[1])
