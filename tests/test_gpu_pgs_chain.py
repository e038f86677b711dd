"""The register chains of the contact solve against the FP64 oracle, where their layout or branches change: the set
sizes around a wave's 64 contacts and the chains' 512, records that need the guarded slip pass, magnitudes at which the
unnormalised slip iterate leaves its range, and pass counts other than the unrolled eight.

Tolerance: a sweep is a contraction whose rounding is that of a few hundred FP64 operations per contact, so forces agree
to 1e-10 relative with identical branches (the bar of the other parity tests)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle.icr_oracle as O  # noqa: E402
from paper_2306_06946_amd.scenes import random_contact_problem  # noqa: E402

pytestmark = pytest.mark.gpu
H = 0.01


def _solve(W, d, mu, lam0, sweeps, j):
    from paper_2306_06946_amd import icr
    s = icr.Scene()
    lam = torch.from_numpy(np.ascontiguousarray(lam0)).cuda()
    st = torch.empty(len(mu), dtype=torch.int8, device="cuda")
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (W.ravel(), d, mu)]
    s.solve_contacts(*dev, H, lam, st, sweeps, 0.0, j)
    return lam.cpu().numpy(), st.cpu().numpy()


def _check(W, d, mu, lam0, sweeps, j=8):
    ref, st_ref, _, _ = O.pgs(W, d, mu, H, lam0, sweeps, 0.0, j)
    print(f"[gpu] pgs nc={len(mu)} sweeps={sweeps} j={j} branches {np.bincount(st_ref, minlength=3)}", flush=True)
    lam, st = _solve(W, d, mu, lam0, sweeps, j)
    assert np.array_equal(st, st_ref)
    assert np.linalg.norm(lam - ref) <= 1e-10 * np.linalg.norm(ref)
    return st_ref


@pytest.mark.parametrize("nc", [1, 2, 3, 5, 63, 64, 65, 66, 127, 128, 129, 193, 512, 513, 700])
def test_set_sizes(nc):
    rng = np.random.default_rng(500 + nc)
    W, d, mu, lam0 = random_contact_problem(nc, rng)
    d[::3] = -np.abs(d[::3])          # every contact pressed at the start: the set has nc contacts
    lam0[::3] = rng.uniform(0.0, 1e-3, nc) * (rng.uniform(size=nc) < 0.5)
    st = _check(W, d, mu, lam0, 6)
    assert nc < 60 or len(set(st.tolist())) == 3


@pytest.mark.parametrize("nc", [40, 150])
@pytest.mark.parametrize("mu_scale", [0.0, 6.0])
def test_friction_beyond_the_fast_slip_pass(nc, mu_scale):
    """mu = 0, and friction so large that w_nn <= mu |w_nt| for most contacts (the guarded pass)."""
    rng = np.random.default_rng(900 + nc)
    W, d, mu, lam0 = random_contact_problem(nc, rng)
    for a in range(nc):               # strongly coupled normal and tangent in each block
        q = np.linalg.qr(rng.standard_normal((3, 3)))[0]
        W[3 * a:3 * a + 3, 3 * a:3 * a + 3] += q @ np.diag([400.0, 40.0, 4.0]) @ q.T
    W = 0.5 * (W + W.T)
    st = _check(W, d, mu * mu_scale, lam0, 3)
    assert 2 in st


@pytest.mark.parametrize("dscale,wscale", [(1e-40, 1e-60), (1e40, 1.0), (1e-20, 1.0)])
def test_magnitudes_beyond_the_unnormalised_iterate(dscale, wscale):
    rng = np.random.default_rng(33)
    W, d, mu, lam0 = random_contact_problem(80, rng)
    _check(W * wscale, d * dscale, mu, lam0, 4)


@pytest.mark.parametrize("j", [0, 1, 7, 20])
@pytest.mark.parametrize("nc", [50, 90, 600])
def test_pass_counts(nc, j):
    rng = np.random.default_rng(700 + nc)
    W, d, mu, lam0 = random_contact_problem(nc, rng)
    _check(W, d, mu, lam0, 3, j)


def test_long_run_of_separated_contacts():
    """Contacts of the set that carry nothing and stay open are passed over, in both the chains and the block sweeps."""
    for nc in (300, 900):
        rng = np.random.default_rng(nc)
        W, d, mu, lam0 = random_contact_problem(nc, rng)
        d[::3] = np.abs(d[::3]) + 1e-4
        d[0:3 * (nc // 8):3] = -1e-3
        lam0 = np.where(np.repeat(rng.uniform(size=nc) < 0.95, 3), 1e-4, 0.0)   # the start set has nearly all contacts
        lam0.reshape(-1, 3)[:, 1:] = 0.0
        _check(W, d, mu, lam0, 4)


@pytest.mark.parametrize("nc", [65, 66, 68, 70, 129, 194, 513, 514, 642])
def test_short_last_block_that_is_passed_over(nc):
    """The last wave's (or block's) few contacts open in the first sweep and are passed over from then on, so that wave
    ends its sweep while the one before it may not have ended its own: the count of solved contacts must not go back (a
    wait for it would run out, and eps be NaN)."""
    rng = np.random.default_rng(40 + nc)
    W, d, mu, lam0 = random_contact_problem(nc, rng)
    last = (nc - 1) // (64 if nc <= 512 else 128) * (64 if nc <= 512 else 128)
    d[::3] = -np.abs(d[::3])
    lam0[::3] = 1e-4
    d[3 * last::3] = 10.0 * np.abs(d).max()
    st = _check(W, d, mu, lam0, 60 if nc <= 512 else 20)
    assert np.all(st[last:] == 0) and np.any(st[:last] != 0)
