"""The FP64 judge where the number of its chunks changes (960 samples), against
the oracle: sums of n terms of one sign to n ulps, forces to the same of the sum
of their terms' magnitudes."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import to_dev
from paper_0909_0541_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s", [1, 960, 961])
@pytest.mark.parametrize("n", [3000, 40000])
def test_chunks(gpu, n, s):
    pos, mass = inputs.uniform_cube(n, 7)[0], np.random.default_rng(n).uniform(0.5, 2.0, n)
    idx = np.random.default_rng(s).integers(0, n, s)
    a_o, p_o = oracle.direct(pos, mass, 1e-2, idx)
    c = gpu.Context()
    a, p = c.direct_sampled(to_dev(pos), to_dev(mass), 1e-2, to_dev(idx, torch.int64))
    d2 = ((pos[None] - pos[idx[:20]][:, None]) ** 2).sum(2) + 1e-4
    scale = (mass / d2).sum(1).max()
    assert np.all(np.abs(p.cpu().numpy() - p_o) <= n * 2.0**-52 * np.abs(p_o))
    assert np.all(np.abs(a.cpu().numpy() - a_o) <= n * 2.0**-52 * scale)
