"""What the timers and the error of a step tell of outlier groups and of walks
that were repeated."""
import numpy as np
import pytest

from gpu_helpers import to_dev
from paper_0909_0541_amd import inputs

pytestmark = pytest.mark.gpu


def _spheres(k, n):
    """Plummer spheres far apart: the outskirts of each have outlier groups."""
    pos = np.concatenate([inputs.plummer(n, s % 4, with_vel=False)[0] + [1e4 * (s % 5), 1e4 * (s // 5), 0.0]
                          for s in range(k)])
    return to_dev(pos), to_dev(np.full(k * n, 1.0 / n)), k * n


def test_walks_of_outliers_are_walk_time(gpu):
    """A wave per group: lots of outliers, whose walks and the waits for them are
    no part of the sums' time (1.33 ms with no group apart, 1.54 with them, 1.93
    with their walks)."""
    pos, mass, n = _spheres(115, 12000)
    force = {}
    for split in (0, -1):
        c = gpu.Context(timing=True, split_visits=split)
        c.build_tree(pos, mass)
        c.make_groups(256)
        t = []
        for k in range(6):
            c.compute_forces(1e-2, 0.8)
            st = c.get_stats()
            assert st.n_force_calls == 1 and st.n_walk_calls == (1 if k else st.n_walk_attempts)
            assert (st.n_split_groups > 64) == (split == 0)
            t.append(st.t_force_ms)
        force[split] = min(t[2:])
    assert force[0] <= 1.3 * force[-1], force


@pytest.mark.parametrize("n,n_crit,theta", [(30000, 64, 0.1), (100000, 256, 0.05)])
@pytest.mark.parametrize("quad", [False, True])
def test_repeated_walks_are_one_force_call(gpu, quad, n, n_crit, theta):
    """Lists longer than the pools hold at first: the walk is counted again, the
    call is not."""
    c = gpu.Context(timing=True, quadrupole=quad)
    c.build_tree(to_dev(inputs.plummer(n, 1, with_vel=False)[0]), to_dev(np.full(n, 1.0 / n)))
    c.make_groups(n_crit)
    for first in (True, False):
        c.compute_forces(1e-2, theta)
        st = c.get_stats()
        assert st.error_flags == 0 and st.n_force_calls == 1
        assert st.n_walk_calls == st.n_walk_attempts and (st.n_walk_calls > 1) == first


def test_replay_names_the_outliers(gpu):
    bh = gpu
    pos, mass, n = _spheres(39, 10000)
    x = to_dev(inputs.uniform_cube(n, 1)[0])
    c = bh.Context()
    c.graph_capture([0, n], x, mass, 256, 1e-2, 1.0)
    x.copy_(pos)
    c.graph_launch()
    with pytest.raises(bh.BHError, match="outlier groups"):
        c.sync()
