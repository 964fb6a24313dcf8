"""A context integrates from its first kick or drift of a particle on: its
quadrupole sums keep the order that one wave sums a list in.  Calls without
particles change nothing."""
import numpy as np
import pytest
import torch

from gpu_helpers import to_dev
from paper_0909_0541_amd import inputs

pytestmark = pytest.mark.gpu


def _forces(c, x, m):
    c.build_tree(x, m)
    c.make_groups(64)
    return [v.clone() for v in c.compute_forces(1e-2, 0.6)]


@pytest.mark.parametrize("call", ["kick", "drift", "leapfrog"])
def test_calls_without_particles(gpu, call):
    n = 5000
    x, m = to_dev(inputs.plummer(n, 1, with_vel=False)[0]), to_dev(np.full(n, 1.0 / n))
    one, two = gpu.Context(quadrupole=True), gpu.Context(quadrupole=True)

    def step(k):
        v = torch.zeros((k, 3), dtype=torch.float64, device=x.device)
        a, p = (torch.zeros(s, dtype=torch.float32, device=x.device) for s in ((k, 3), (k,)))
        if call == "kick":
            two.kick(v, a, 0.0)
        elif call == "drift":
            two.drift(x[:k].clone(), v, 0.0)
        else:
            two.leapfrog(x[:k].clone(), v, m[:k].contiguous(), 1e-2, 0.6, 64, 0.0, 1, a, p)

    before = _forces(one, x, m)
    step(0)
    assert all(torch.equal(s, t) for s, t in zip(before, _forces(two, x, m)))
    step(100)
    after = _forces(two, x, m)
    assert not torch.equal(before[0], after[0])
    # FP32 sums of the same entries in two orders
    assert float(((before[0] - after[0]).norm(dim=1) / before[0].norm(dim=1).mean()).max()) <= 1e-5
