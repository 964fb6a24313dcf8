"""Neighbour search where most candidates are neighbours (radii that cover much of
the system), the members testing their candidates one after another, beside
sparse places of the same call.  Counts and lists equal, densities to 1e-12 of
theirs (n terms of one sign, each a few roundings from the kernel's value),
against all pairs in plain FP64."""
import numpy as np
import pytest
import torch

from gpu_helpers import to_dev
from paper_0909_0541_amd import inputs

pytestmark = pytest.mark.gpu


def _reference(x, m, h):
    """Counts and densities of all pairs, by rows."""
    n = x.shape[0]
    count = torch.zeros(n, dtype=torch.int32, device=x.device)
    rho = torch.zeros(n, dtype=torch.float64, device=x.device)
    rows = []
    for a in range(0, n, 1000):
        d = x[None, :, :] - x[a:a + 1000, None, :]
        r2 = (d[..., 0] * d[..., 0] + d[..., 1] * d[..., 1]) + d[..., 2] * d[..., 2]
        hh = h[a:a + 1000, None]
        near = r2 < hh * hh
        near[torch.arange(near.shape[0]), torch.arange(a, a + near.shape[0])] = False
        q = r2.sqrt() / hh
        w = torch.where(q < 0.5, 1 - 6 * q * q + 6 * q * q * q, 2 * (1 - q).clamp_min(0) ** 3)
        s = 8 / (np.pi * h[a:a + 1000] ** 3)
        count[a:a + 1000] = near.sum(1, dtype=torch.int32)
        rho[a:a + 1000] = m[a:a + 1000] * s + s * torch.where(near, m[None, :] * w, torch.zeros_like(w)).sum(1)
        rows.append(near)
    return count, rho, rows


@pytest.mark.parametrize("radii", ["all", "half", "mixed", "tiny", "huge"])
@pytest.mark.parametrize("n,n_crit", [(2, 1), (65, 64), (700, 1), (3000, 8), (3000, 63), (3000, 64), (3000, 65), (5000, 200),
                                      (9000, 64), (9000, 256)])
def test_dense(gpu, n, n_crit, radii):
    pos = inputs.clustered(n, 6, n_halos=2)[0] if n > 65 else inputs.uniform_cube(n, 3)[0]
    scale = {"tiny": 1e-130, "huge": 1e130}.get(radii, 1.0)  # (radii beyond 2^400: the other quotient)
    rng = np.random.default_rng(n)
    h = {"all": np.full(n, 2.5), "half": np.full(n, 0.05)}.get(radii, rng.choice([0.01, 0.1, 2.5], n)) * scale
    x, m, h = to_dev(pos * scale), to_dev(rng.uniform(0.5, 1.5, n)), to_dev(h)
    if radii in ("tiny", "huge"):  # (the kernel's normalisation would leave FP64's range: counts only)
        ref = _reference(x / scale, m, h / scale)[0]
    else:
        ref, rho_ref, rows = _reference(x, m, h)
    c = gpu.Context()
    c.build_tree(x, m)
    c.make_groups(n_crit)
    count, _ = c.neighbors(h)
    c.sync()
    if radii in ("tiny", "huge"):
        # (scaled by other than a power of two: a pair in 10^6 may fall on the other side)
        assert int((count - ref).abs().sum()) <= 1e-6 * n * n
        return
    assert torch.equal(count, ref)
    count, rho = c.neighbors(h, rho=True)
    assert torch.equal(count, ref)
    assert float(((rho - rho_ref).abs() / rho_ref).max()) <= 1e-12
    off, nbr = c.neighbor_lists(h)
    c.sync()
    assert torch.equal(off[1:] - off[:-1], ref.long())
    who = torch.repeat_interleave(torch.arange(n, device="cuda"), ref.long())
    order = torch.argsort(who * n + nbr.long())
    assert torch.equal(nbr[order].long(), torch.cat([r.nonzero()[:, 1] for r in rows]))
