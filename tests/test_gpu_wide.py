"""The workgroup walk with list blocks (quadrupoles, default options, up to 2048
n_crit particles), the sums by tiles (the same without quadrupoles) and the
outliers' walk tasks (both below and above that size), against the FP64 oracle: list lengths and interaction counts exactly, forces to
the parity bar, list masses to the bound of two orders of one FP64 sum.

Sizes sit at the edges of the path: member blocks of 64 (64/65, 128/129, 256),
the smallest group size that takes it, trees of 1 to 3 particles, list blocks
just filled, cells whose children are many coincident particles, groups whose
lists are the whole system (outliers: some, and at theta = 0 every group, more
than there is room for), a pool that has to grow, and the largest tree of the
path beside the smallest that does not take it.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import check_forces, gpu_run, to_dev
from paper_0909_0541_amd import inputs

pytestmark = pytest.mark.gpu


def _check(bh, pos, mass, eps, theta, n_crit, **opts):
    c = bh.Context(**opts)
    c, acc, pot, st, G = gpu_run(bh, pos, mass, eps, theta, n_crit, ctx=c)
    assert st.error_flags == 0
    t = oracle.Tree(pos, mass, curve=opts.get("curve", 0))
    assert t.groups(n_crit) == G
    ref = t.forces(eps, theta, quadrupole=opts.get("quadrupole", False))
    _, _, ll, lm = c.export_groups(lists=True)
    ll, lm = ll.cpu().numpy(), lm.cpu().numpy()
    assert np.array_equal(ll, ref["list_len"])
    assert np.all(np.abs(lm - ref["list_mass"]) <= 2.0 * np.maximum(ll - 1, 0) * 2.0**-53 * ref["list_mass"])
    assert st.interactions == ref["interactions"] and st.max_list == ll.max() and st.list_entries == ll.sum()
    check_forces(acc, pot, ref)
    return c, st


@pytest.mark.parametrize("n", [1, 2, 3, 255, 256, 257, 1000])
@pytest.mark.parametrize("n_crit", [16, 64, 256])
@pytest.mark.parametrize("quad", [False, True])
def test_small_trees(gpu, n, n_crit, quad):
    pos, mass = inputs.uniform_cube(n, 3 + n)[:2]
    _check(gpu, pos, mass, 1e-2, 0.6, n_crit, quadrupole=quad)


@pytest.mark.parametrize("n_crit", [16, 63, 64, 65, 128, 129, 200, 256])
@pytest.mark.parametrize("quad", [False, True])
def test_member_blocks(gpu, n_crit, quad):
    pos, mass = inputs.clustered(6000, 11, n_halos=5)[:2]
    _check(gpu, pos, mass, 1e-4, 0.6, n_crit, quadrupole=quad)


@pytest.mark.parametrize("quad,curve", [(True, 0), (True, 1), (False, 1)])
def test_options(gpu, quad, curve):
    pos, mass = inputs.clustered(20000, 12, n_halos=10)[:2]
    _check(gpu, pos, mass, 1e-3, 0.6, 128, quadrupole=quad, curve=curve)


def test_buckets_of_many_coincident_particles(gpu):
    """Cells with more than eight children (equal keys), more of them than a
    workgroup's threads, in and out of other groups' reach."""
    rng = np.random.default_rng(5)
    pos = np.concatenate([np.repeat(rng.uniform(0, 1, (40, 3)), 70, axis=0), np.repeat([[0.3, 0.3, 0.3]], 2500, axis=0),
                          rng.uniform(0, 1, (1500, 3))])
    _check(gpu, pos, np.full(len(pos), 1.0 / len(pos)), 1e-2, 0.5, 64)


def _spread(n, seed=1):
    """A ball inside one octant of the cube and one particle in each of the
    others: those seven are one group whose box covers the ball, so its list is
    every particle."""
    pos, mass = inputs.uniform_sphere(n - 7, seed)[:2]
    corners = np.array([[x, y, z] for x in (0.0, 1.0) for y in (0.0, 1.0) for z in (0.0, 1.0)])[:7]
    pos = np.concatenate([corners, 0.7 + 0.1 * pos])
    pos[-1] = 1.0
    return pos, np.full(n, 1.0 / n)


@pytest.mark.parametrize("n,n_crit", [(3000, 16), (9000, 64), (40000, 256), (40000, 16)])
@pytest.mark.parametrize("quad", [False, True])
def test_outliers(gpu, n, n_crit, quad):
    """At n_crit 16 and 40000 particles the ordinary groups are walked by single
    waves; 3000 particles have no walk long enough to be given up."""
    pos, mass = _spread(n)
    _, st = _check(gpu, pos, mass, 1.0 / 256, 0.75, n_crit, quadrupole=quad)
    assert st.max_list == n
    if n > 3000:
        assert 1 <= st.n_split_groups <= 160 and st.n_segments > st.n_split_groups


def test_theta_zero_has_no_outliers(gpu):
    """theta = 0: every list is the whole system, which is then ordinary."""
    pos, mass = inputs.uniform_sphere(12000, 8)[:2]
    _, st = _check(gpu, pos, mass, 1e-2, 0.0, 16)
    assert st.max_list == 12000 and st.n_split_groups == 0


def test_more_outliers_than_places(gpu):
    """300 groups that span the whole of their systems (a batch of 300 balls as
    in _spread): with more than 256 outliers every group is walked whole, in a
    captured step too."""
    bh = gpu
    pos, mass = _spread(9000, 2)
    k = 300
    off = np.arange(k + 1, dtype=np.int64) * 9000
    dpos, dmass = to_dev(np.tile(pos, (k, 1))), to_dev(np.tile(mass, k))
    t = oracle.Tree(pos, mass)
    t.groups(64)
    ref = t.forces(1e-2, 0.8)
    c = bh.Context()
    acc, pot = c.graph_capture(off, dpos, dmass, 64, [1e-2] * k, [0.8] * k)
    for _ in range(2):
        st = c.get_stats()
        assert st.error_flags == 0 and st.n_split_groups == 0
        assert st.interactions == k * int(ref["interactions"])
        for s in (0, 150, 299):
            check_forces(acc[9000 * s:9000 * (s + 1)].cpu().numpy().astype(np.float64),
                         pot[9000 * s:9000 * (s + 1)].cpu().numpy().astype(np.float64), ref)
        acc.zero_()
        c.graph_launch()
        c.sync()


def test_outliers_in_a_batch(gpu):
    bh = gpu
    parts = [_spread(k, 50 + k) for k in (20000, 8, 17000, 9, 9000)]
    pos, mass = (np.concatenate([p[k] for p in parts]) for k in range(2))
    off = np.concatenate([[0], np.cumsum([len(p[0]) for p in parts])])
    for n_crit in (16, 64):
        c = bh.Context()
        c.build_batch(off, to_dev(pos), to_dev(mass))
        c.make_groups(n_crit)
        acc, pot = c.compute_forces_batch([1e-2] * 5, [0.7] * 5)
        st = c.get_stats()
        assert st.error_flags == 0 and st.n_split_groups > 0
        acc, pot = acc.cpu().numpy().astype(np.float64), pot.cpu().numpy().astype(np.float64)
        inter = 0
        for k in range(5):
            a, b = off[k], off[k + 1]
            t = oracle.Tree(pos[a:b], mass[a:b])
            t.groups(n_crit)
            ref = t.forces(1e-2, 0.7)
            inter += int(ref["interactions"])
            check_forces(acc[a:b], pot[a:b], ref)
        assert st.interactions == inter


@pytest.mark.parametrize("n,n_crit", [(9000, 64), (40000, 16)])
@pytest.mark.parametrize("quad", [False, True])
def test_replays_and_repeats_agree(gpu, n, n_crit, quad):
    """Outliers included: eager calls and graph replays, with other work on the
    context's buffers between them, give the same bits."""
    bh = gpu
    pos, mass = _spread(n, 4)
    dpos, dmass = to_dev(pos), to_dev(mass)
    e = bh.Context(quadrupole=quad)
    a0, p0 = bh.tree_forces(dpos, dmass, 1e-2, 0.7, n_crit, ctx=e)
    a1, p1 = bh.tree_forces(dpos, dmass, 1e-2, 0.7, n_crit, ctx=e)
    assert torch.equal(a0, a1) and torch.equal(p0, p1)
    a2, p2 = e.compute_forces(1e-2, 0.7)  # the same tree and groups again
    assert torch.equal(a0, a2) and torch.equal(p0, p2)
    c = bh.Context(quadrupole=quad)
    acc, pot = c.graph_capture([0, n], dpos, dmass, n_crit, [1e-2], [0.7])
    for _ in range(3):
        acc.zero_()
        pot.zero_()
        c.graph_launch()
        c.sync()
        assert torch.equal(acc, a0) and torch.equal(pot, p0)
        bh.tree_forces(dpos[: n // 2].contiguous(), dmass[: n // 2].contiguous(), 1e-2, 0.7, n_crit, ctx=e)
        torch.cuda.synchronize()


@pytest.mark.parametrize("quad", [False, True])
def test_block_pool_grows(gpu, quad):
    """Lists far longer than the first estimate (theta small): the walk is run
    again, with the same result as a second call's."""
    bh = gpu
    pos, mass = inputs.clustered(60000, 21, n_halos=30)[:2]
    c = bh.Context(quadrupole=quad)
    c.build_tree(to_dev(pos), to_dev(mass))
    c.make_groups(64)
    a1, p1 = (v.clone() for v in c.compute_forces(1e-4, 0.15))
    assert c.get_stats().n_walk_attempts >= 2
    a2, p2 = c.compute_forces(1e-4, 0.15)
    assert c.get_stats().n_walk_attempts == 1
    assert torch.equal(a1, a2) and torch.equal(p1, p2)
    t = oracle.Tree(pos, mass)
    t.groups(64)
    check_forces(a1.cpu().numpy().astype(np.float64), p1.cpu().numpy().astype(np.float64), t.forces(1e-4, 0.15, quadrupole=quad))


def test_path_boundary(gpu):
    """2048 n_crit particles and one more: the two paths' lists are the same."""
    for n in (2048 * 16, 2048 * 16 + 1):
        pos, mass = inputs.clustered(n, 6, n_halos=16)[:2]
        _check(gpu, pos, mass, 1e-4, 0.7, 16)
