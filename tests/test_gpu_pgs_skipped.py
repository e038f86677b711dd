"""Active-set PGS with contacts outside the set whose gaps the bound cannot settle: every sweep's skipped contacts must be
verified from the running reference state, and one that closes late must join the set.  The oracle sweeps all contacts.

Forces agree to 1e-10 relative with identical branches (the bar of the other parity tests)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle.icr_oracle as O  # noqa: E402
from paper_2306_06946_amd.scenes import random_spd  # noqa: E402

pytestmark = pytest.mark.gpu


def _problem(nc, share, margin, off, seed):
    """Gaps with a known solution: `share` of the contacts pressed, the others open by `margin` times the motion that the
    forces cause (some closed by the warm start, which is `off` from the solution)."""
    rng = np.random.default_rng(seed)
    W = random_spd(3 * nc, rng)
    mu = rng.uniform(0.2, 0.6, nc)
    on = rng.uniform(size=nc) < share
    ln = rng.uniform(0.2, 1.8, nc) * on
    ang = rng.uniform(0, 2 * np.pi, nc)
    lt = (mu * ln * rng.uniform(0, 1.0, nc))[:, None] * np.stack([np.cos(ang), np.sin(ang)], 1)
    lam = np.concatenate([ln[:, None], lt], 1)
    h = 0.01
    move = (h * h) * (W @ lam.ravel()).reshape(nc, 3)
    d = -move
    d[:, 0] += np.where(on, 0.0, margin * np.abs(move).max() * rng.uniform(1e-3, 1.0, nc))
    return W, d.ravel(), mu, (lam * rng.uniform(1 - off, 1 + off, nc)[:, None]).ravel(), h


@pytest.mark.parametrize("nc,share", [(6, 0.5), (65, 0.1), (150, 0.3), (300, 0.12), (300, 0.7), (600, 0.1), (1100, 0.05)])
@pytest.mark.parametrize("margin,off", [(0.05, 0.2), (0.002, 0.6)])
def test_skipped_contacts(nc, share, margin, off):
    from paper_2306_06946_amd import icr
    W, d, mu, lam0, h = _problem(nc, share, margin, off, 11)
    print(f"[gpu] skipped {nc} {share} {margin} {off}", flush=True)
    sweeps = 12
    ref = O.pgs(W, d, mu, h, lam0, sweeps, 0.0, 8)
    g = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (W, d, mu, lam0)]
    lam = g[3].clone()
    status = torch.zeros(nc, dtype=torch.int8, device="cuda")
    s = icr.Scene()
    n, _ = s.solve_contacts(g[0], g[1], g[2], h, lam, status, sweeps, 0.0)
    assert n == ref[2]
    got = lam.cpu().numpy()
    assert np.linalg.norm(got - ref[0].ravel()) <= 1e-10 * np.linalg.norm(ref[0])
    assert np.array_equal(status.cpu().numpy(), ref[1])
