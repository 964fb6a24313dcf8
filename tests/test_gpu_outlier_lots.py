"""More outlier groups than are walked and summed together (256): they come in
lots, eager and captured, at sizes summed by tiles and by a wave per group.
Against the FP64 oracle system by system; repeats and replays bit for bit."""
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


@pytest.mark.parametrize("k,n,n_crit,lots", [(100, 5000, 256, 2), (120, 30000, 256, 2)])
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


def test_replay_with_more_than_recorded(gpu):
    """A step captured on systems without outliers and replayed on systems with
    hundreds reports it; captured again, it has room."""
    bh = gpu
    k, n = 100, 5000
    _, pos, mass, off = _batch(k, n)
    plain = to_dev(np.tile(inputs.uniform_cube(n, 1)[0], (k, 1)))
    c = bh.Context()
    c.graph_capture(off, plain, mass, 256, 1e-2, 0.8)
    assert c.get_stats().n_split_groups == 0
    plain.copy_(pos)
    c.graph_launch()
    with pytest.raises(bh.BHError):
        c.sync()
    acc, pot = c.graph_capture(off, plain, mass, 256, 1e-2, 0.8)
    c.build_batch(off, pos, mass)
    c.make_groups(256)
    a, p = c.compute_forces_batch([1e-2] * k, [0.8] * k)
    acc.zero_()
    c.graph_launch()
    c.sync()
    assert torch.equal(acc, a) and torch.equal(pot, p)
