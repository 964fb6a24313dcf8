"""More outlier groups than are walked and summed together (256, or 64 in a single
system of up to 400,000 particles): they come in lots, eager and captured, at
sizes summed by tiles and by a wave per group.  Against the FP64 oracle system by system, or against
whole walks; repeats and replays bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import check_forces, to_dev
from paper_0909_0541_amd import inputs

pytestmark = pytest.mark.gpu


def _batch(k, n):
    # (four different systems in turn)
    one = [inputs.plummer(n, s, with_vel=False)[0] for s in range(4)]
    pos = np.concatenate([one[s % 4] for s in range(k)])
    return one, to_dev(pos), to_dev(np.full(k * n, 1.0 / n)), np.arange(k + 1, dtype=np.int64) * n


@pytest.mark.parametrize("k,n,n_crit,lots", [(120, 30000, 256, 2)])
def test_lots(gpu, k, n, n_crit, lots):
    bh = gpu
    one, pos, mass, off = _batch(k, n)
    eps, theta = 1e-2, 0.8
    c = bh.Context()
    c.build_batch(off, pos, mass)
    c.make_groups(n_crit)
    a, p = (v.clone() for v in c.compute_forces_batch([eps] * k, [theta] * k))
    st = c.get_stats()
    assert st.error_flags == 0 and (lots - 1) * 256 < st.n_split_groups <= lots * 256
    _, _, ll, _ = c.export_groups(lists=True)
    inter = 0
    for s in range(4):
        t = oracle.Tree(one[s], np.full(n, 1.0 / n))
        t.groups(n_crit)
        ref = t.forces(eps, theta)
        inter += int(ref["interactions"]) * len(range(s, k, 4))
        check_forces(a[s * n:(s + 1) * n].cpu().numpy().astype(np.float64),
                     p[s * n:(s + 1) * n].cpu().numpy().astype(np.float64), ref)
        # the same system elsewhere in the batch, whichever lot its outliers were in
        for j in range(s + 4, k, 4):
            assert torch.equal(a[j * n:(j + 1) * n], a[s * n:(s + 1) * n]), (s, j)
    assert st.interactions == inter and st.max_list == int(ll.max()) == n
    b, q = c.compute_forces_batch([eps] * k, [theta] * k)
    assert torch.equal(a, b) and torch.equal(p, q)
    assert c.get_stats().n_split_groups == st.n_split_groups and c.get_stats().n_segments == st.n_segments
    g = bh.Context()
    acc, pot = g.graph_capture(off, pos, mass, n_crit, eps, theta)
    for _ in range(2):
        acc.zero_()
        g.graph_launch()
        g.sync()
        assert torch.equal(acc, a) and torch.equal(pot, p)
        assert g.get_stats().n_split_groups == st.n_split_groups


def _spheres(k, n):
    """Plummer spheres far apart in one system: the outskirts of each are
    a few groups whose lists hold nearly all of it."""
    pos = np.concatenate([inputs.plummer(n, s % 4, with_vel=False)[0] + [1e4 * (s % 5), 1e4 * (s // 5), 0.0]
                          for s in range(k)])
    return to_dev(pos), to_dev(np.full(k * n, 1.0 / n)), k * n


@pytest.mark.parametrize("k,n,theta", [(39, 10000, 1.0), (70, 20000, 0.8), (110, 14000, 0.8)])
def test_single_system(gpu, k, n, theta):
    bh = gpu
    pos, mass, n = _spheres(k, n)
    res = []
    for opts in ({}, {"split_visits": -1}):
        c = bh.Context(**opts)
        c.build_tree(pos, mass)
        c.make_groups(256)
        a, p = (v.clone() for v in c.compute_forces(1e-2, theta))
        b, q = c.compute_forces(1e-2, theta)
        assert torch.equal(a, b) and torch.equal(p, q)
        res.append((a, p, c.get_stats(), c.export_groups(lists=True)[2]))
    (a, p, st, ll), (b, q, whole, ll_whole) = res
    assert st.error_flags == 0 and 64 < st.n_split_groups <= 320 and whole.n_split_groups == 0
    assert (st.n_split_groups > 256) == (k > 100)
    assert torch.equal(ll, ll_whole) and st.interactions == whole.interactions
    # FP32 sums of the same entries in two orders
    assert float(((a - b).norm(dim=1) / (b.norm(dim=1) + b.norm(dim=1).mean())).max()) <= 1e-5
    assert float(((p - q).abs() / q.abs()).max()) <= 1e-5
    g = bh.Context()
    acc, pot = g.graph_capture([0, n], pos, mass, 256, 1e-2, theta)
    for _ in range(3):
        acc.zero_()
        g.graph_launch()
        g.sync()
        assert torch.equal(acc, a) and torch.equal(pot, p)
        assert g.get_stats().n_split_groups == st.n_split_groups


def test_replay_with_more_than_recorded(gpu):
    """A step captured on a system without outliers and replayed on one with
    more than a lot reports it; captured again, it has room."""
    bh = gpu
    pos, mass, n = _spheres(39, 10000)
    x = to_dev(inputs.uniform_cube(n, 1)[0])
    c = bh.Context()
    c.graph_capture([0, n], x, mass, 256, 1e-2, 1.0)
    assert c.get_stats().n_split_groups == 0
    x.copy_(pos)
    c.graph_launch()
    with pytest.raises(bh.BHError):
        c.sync()
    acc, pot = c.graph_capture([0, n], x, mass, 256, 1e-2, 1.0)
    c.build_tree(pos, mass)
    c.make_groups(256)
    a, p = c.compute_forces(1e-2, 1.0)
    acc.zero_()
    c.graph_launch()
    c.sync()
    assert torch.equal(acc, a) and torch.equal(pot, p)
