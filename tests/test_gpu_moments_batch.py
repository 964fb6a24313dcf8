"""Moments of batches of many systems (from 256 on the subtrees of at most 64
particles have launches of their own), by the size of the largest system: 64, 512
and 1024 are the limits of the subtrees, and of what else is launched.  Every
system's node records and second moments bit for bit those of a tree of its own."""
import numpy as np
import pytest
import torch

from gpu_helpers import to_dev
from paper_0909_0541_amd import inputs

pytestmark = pytest.mark.gpu


def _system(n):
    rng = np.random.default_rng(n)
    pos = inputs.clustered(n, 3, n_halos=2)[0] if n > 600 else rng.uniform(-1.0, 1.0, (n, 3))
    if n > 8:
        pos[: n // 4] = pos[0]  # a bucket
    return pos, rng.uniform(0.5, 1.5, n)


def _records(ints, reals, mom, i, first, count):
    """Rows i sorted by particle range, as one array."""
    key = (ints[i, 2] - first).long() * (count + 1) + ints[i, 3]
    i = i[key.argsort(stable=True)]
    rows = [ints[i, 1:2].double(), (ints[i, 2:3] - first).double(), ints[i, 3:4].double(), reals[i]]
    return torch.cat(rows + ([mom[i]] if mom is not None else []), 1)


@pytest.mark.parametrize("quad", [False, True])
@pytest.mark.parametrize("systems", [255, 256, 700])
@pytest.mark.parametrize("sizes", [(1, 2, 0, 5), (63, 64, 1, 0), (65, 3, 64), (511, 512, 2, 40), (513, 7), (1023, 1024, 64, 0),
                                   (1025, 33), (5000, 1, 2, 3, 4, 5, 6, 7)])
def test_batches(gpu, sizes, systems, quad):
    n_sys = [sizes[k % len(sizes)] for k in range(systems)]
    off = np.concatenate([[0], np.cumsum(n_sys)])
    one = {n: _system(n) for n in sizes if n}
    b = gpu.Context(quadrupole=quad)
    b.build_batch(off, to_dev(np.concatenate([one[n][0] for n in n_sys if n])),
                  to_dev(np.concatenate([one[n][1] for n in n_sys if n])))
    ints, reals = b.export_nodes()
    mom = b.export_moments() if quad else None
    assert b.get_stats().error_flags == 0
    for n, (pos, mass) in one.items():
        c = gpu.Context(quadrupole=quad)
        c.build_tree(to_dev(pos), to_dev(mass))
        i1, r1 = c.export_nodes()
        want = _records(i1, r1, c.export_moments() if quad else None, torch.arange(len(i1), device=i1.device), 0, n)
        of_size = [s for s in range(systems) if n_sys[s] == n]
        for s in (of_size[0], of_size[len(of_size) // 2], of_size[-1]):
            f = int(off[s])
            # (kind 3: roots of empty systems)
            i = ((ints[:, 1] != 3) & (ints[:, 2] >= f) & (ints[:, 2] + ints[:, 3] <= f + n)).nonzero()[:, 0]
            assert torch.equal(_records(ints, reals, mom, i, f, n), want), (n, s)
