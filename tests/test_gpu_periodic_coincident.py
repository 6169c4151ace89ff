"""Periodic potential of particles at exactly the same place: the pair's limit, softened
1 / eps less the smooth part's value at r = 0, in every kind of item (the same piece
of a part, other pieces, other parts; one-sided and pair items)."""
import numpy as np
import pytest

import oracle
from paper_1208_3444_amd import colatus, inputs
from conftest import to_dev

pytestmark = pytest.mark.gpu


def _cloud(N):
    x, m = inputs.random_cloud(N, 30 + N, scale=1.6)
    m = m * np.random.default_rng(N).uniform(0.5, 1.5, N)
    # (kept, moved onto it): neighbours, one piece apart, one part apart, first and last
    pairs = [(3, 4)] + [(a, b) for a, b in ((5, 70), (6, 300), (0, N - 1)) if b < N]
    for a, b in pairs:
        x[:, b] = x[:, a]
    return x, m, np.unique(np.array(pairs + [(1, 2)]).ravel())


@pytest.mark.parametrize("prec", ["fp64", "mixed_twosum", "mixed_f64acc", "fp32"])
@pytest.mark.parametrize("N", [6, 200, 1500, 7425, 10753])
def test_coincident_particles(dev, N, prec):
    """Against the oracle, relative to the sums of the pair magnitudes, the
    repository's bars for periodic potentials: 1e-12, and 1e-4 with FP32 pairs."""
    L, eps, G = 1.6, 0.05, 1.2
    x, m, t = _cloud(N)
    _, ref = oracle.forces_periodic(x, m, eps, L, G=G, targets=t, with_phi=True)
    _, phi = colatus.forces_periodic(to_dev(x, dev), to_dev(m, dev), eps, L, G=G, precision=prec,
                                     with_phi=True)
    d = x[:, None, :] - x[:, t][:, :, None]
    d -= L * np.rint(d / L)
    ps = G * (m[None, :] / np.sqrt((d ** 2).sum(axis=0) + eps * eps)).sum(axis=1)
    e = np.abs(phi.cpu().numpy()[t] - ref) / ps
    print(f"N={N} {prec}: {e.max():.2e}", flush=True)
    assert e.max() <= (1e-12 if prec == "fp64" else 1e-4)


@pytest.mark.parametrize("N", [6, 1500])
def test_without_softening_no_splitting_shows(dev, N):
    """eps = 0: the infinite 1 / r left out, the rest does not depend on where the
    sum is split (the window of FP64 pairs, the Gaussian of FP32 pairs)."""
    x, m, t = _cloud(N)
    a, b = (colatus.forces_periodic(to_dev(x, dev), to_dev(m, dev), 0.0, 1.6, precision=p,
                                    with_phi=True)[1].cpu().numpy()[t]
            for p in ("fp64", "mixed_twosum"))
    d = x[:, None, :] - x[:, t][:, :, None]
    d -= 1.6 * np.rint(d / 1.6)
    r2 = (d ** 2).sum(axis=0)
    ps = (m[None, :] / np.sqrt(np.where(r2 == 0.0, np.inf, r2))).sum(axis=1)
    assert np.abs(a - b).max() <= 1e-4 * ps.max()
