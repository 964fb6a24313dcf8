"""Neighbour search without lists (particles of small cells read as runs)
against the search that writes lists (every leaf visited): clumps of particles
on both sides of the run length (256), of a wave and of a matrix tile; radii and
scales beyond the ordinary range of the kernel's quotient.  The same candidates,
so equal counts and statistics; densities to 1e-13 (a few hundred FP64 terms
added in another order: some 1e2 x 1.1e-16)."""
import numpy as np
import pytest
import torch

from gpu_helpers import to_dev
from paper_0909_0541_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_crit", [1, 15, 16, 17, 48, 64, 65, 128, 129, 256])
@pytest.mark.parametrize("power", [-430, 0, 430])
def test_runs_equal_leaves(gpu, n_crit, power):
    rng = np.random.default_rng(n_crit)
    parts = []
    for size in (1, 2, 15, 16, 17, 63, 64, 65, 255, 256, 257, 600):
        centre = rng.uniform(-1.0, 1.0, 3)
        parts.append(centre + rng.uniform(-0.01, 0.01, (size, 3)))
    parts.append(np.tile([[0.3, 0.2, -0.4]], (300, 1)))  # one point
    pos = np.ldexp(rng.permutation(np.concatenate(parts)), power)
    n = pos.shape[0]
    mass = rng.uniform(0.5, 2.0, n)
    h = np.ldexp(np.exp(rng.uniform(np.log(1e-3), np.log(0.5), n)), power)
    c = gpu.Context()
    c.build_tree(to_dev(pos), to_dev(mass))
    c.make_groups(n_crit)
    dh = to_dev(h)
    cnt, rho = c.neighbors(dh, count=True, rho=True)
    s = c.get_stats()
    off = torch.zeros(n + 1, dtype=torch.int64, device=dh.device)
    off[1:] = torch.cumsum(cnt, 0)
    nbr = torch.zeros(int(off[-1]), dtype=torch.int32, device=dh.device)
    cnt2, rho2 = c.neighbors(dh, count=True, rho=True, offsets=off, nbr=nbr)
    r = c.get_stats()
    assert s.error_flags == 0 and r.error_flags == 0
    assert torch.equal(cnt, cnt2) and int(cnt.max()) > 299
    assert s.neighbor_pairs == r.neighbor_pairs and s.neighbor_tests == r.neighbor_tests
    if power == 0:
        assert float(((rho - rho2).abs() / rho2).max()) <= 1e-13


@pytest.mark.parametrize("case", ["plummer", "plummer wide", "all", "batch"])
def test_outliers_equal_lists(gpu, case):
    """Groups whose search takes in thousands of particles (a Plummer sphere's
    outskirts; every group of a box searched at half its side) go to the
    launch by parts; two runs agree bit for bit."""
    rng = np.random.default_rng(3)
    off = None
    if case == "all":
        pos = rng.uniform(-1.0, 1.0, (12000, 3))
        h = np.full(12000, 1.0)
    else:
        sizes = [30000] if case == "plummer" else [100000] if case == "plummer wide" else [9000, 0, 1, 20000]
        pos = np.concatenate([inputs.plummer(k, 5, with_vel=False)[0] if k else np.zeros((0, 3)) for k in sizes])
        r2 = 1.0 + (pos * pos).sum(1)
        h = 0.7 * (3 * 40.0 / (4 * np.pi * 20000)) ** (1.0 / 3.0) * r2 ** (5.0 / 6.0)
        off = np.concatenate([[0], np.cumsum(sizes)])
    n = pos.shape[0]
    mass = rng.uniform(0.5, 2.0, n)
    c = gpu.Context()
    if case == "batch":
        c.build_batch(off, to_dev(pos), to_dev(mass))
    else:
        c.build_tree(to_dev(pos), to_dev(mass))
    c.make_groups(128 if case == "plummer wide" else 64)
    dh = to_dev(h)
    cnt, rho = c.neighbors(dh, count=True, rho=True)
    s = c.get_stats()
    again, rho_again = c.neighbors(dh, count=True, rho=True)
    assert torch.equal(cnt, again) and torch.equal(rho, rho_again)
    off = torch.zeros(n + 1, dtype=torch.int64, device=dh.device)
    off[1:] = torch.cumsum(cnt, 0)
    nbr = torch.zeros(int(off[-1]), dtype=torch.int32, device=dh.device)
    cnt2, rho2 = c.neighbors(dh, count=True, rho=True, offsets=off, nbr=nbr)
    r = c.get_stats()
    assert s.error_flags == 0 and r.error_flags == 0
    assert torch.equal(cnt, cnt2)
    assert s.neighbor_pairs == r.neighbor_pairs and s.neighbor_tests == r.neighbor_tests
    # up to 12,000 terms of one sign in another order: 12,000 x 1.1e-16
    assert float(((rho - rho2).abs() / rho2).max()) <= 1.4e-12
