"""The reciprocal-space kernels and the FP64 splitting of the periodic sum at
the edges of their tiles: 32-particle phase tiles and chunks of the structure
factors, 128-particle blocks and column ranges of the field, the switch of the
FP64 pairs between one-sided and pair items (28 parts of 256 / 30 parts), boxes
whose parts do and do not span half the box, a large softening."""
import numpy as np
import pytest

import oracle
from paper_1208_3444_amd import colatus, inputs
from conftest import to_dev

pytestmark = pytest.mark.gpu


def _scales(x, m, t, L, eps):
    d = x[:, None, :] - x[:, t][:, :, None]
    d -= L * np.rint(d / L)
    r2 = (d ** 2).sum(axis=0)
    r2[np.arange(len(t)), t] = np.inf
    return ((m[None, :] / (r2 + eps * eps)).sum(axis=1),
            (m[None, :] / np.sqrt(r2 + eps * eps)).sum(axis=1))


@pytest.mark.parametrize("N,order,eps", [(31, "random", 0.02), (32, "random", 0.02),
                                         (33, "random", 0.3), (127, "random", 0.02),
                                         (129, "random", 0.0), (7168, "random", 0.004),
                                         (7425, "morton", 0.004), (8193, "random", 0.2)])
def test_fp64_periodic_field_and_potential(dev, N, order, eps):
    """Field and potential of sampled particles against the oracle, relative
    to the sums of the pair magnitudes: FP64 sums of N terms and truncations
    of 1e-15 leave a few 1e-16 times sqrt(N); the bar is the repository's
    1e-12."""
    L, G, a = 1.6, 1.1, 0.9
    if order == "random":
        x, m = inputs.random_cloud(N, 40 + N, scale=L)
    else:
        w = inputs.lcdm_grf(20)
        x, m = np.ascontiguousarray(w.x[:, :N]) * L, w.m[:N] * 1.0
    t = np.sort(np.random.default_rng(N).choice(N, min(N, 96), replace=False))
    ref = oracle.forces_periodic(x, m, eps, L, G=G, a=a, targets=t)
    acc, phi = colatus.forces_periodic(to_dev(x, dev), to_dev(m, dev), eps, L, G=G, a=a,
                                       precision="fp64", with_phi=True)
    acc0 = colatus.forces_periodic(to_dev(x, dev), to_dev(m, dev), eps, L, G=G, a=a,
                                   precision="fp64")
    fs, ps = _scales(x, m, t, L, eps)
    got = acc.cpu().numpy()[:, t]
    e = np.linalg.norm(got - ref, axis=0) / (G / a ** 3 * fs)
    e0 = np.linalg.norm(acc0.cpu().numpy()[:, t] - ref, axis=0) / (G / a ** 3 * fs)
    print(f"N={N} {order}: field {e.max():.2e} / without potential {e0.max():.2e}", flush=True)
    assert e.max() <= 1e-12 and e0.max() <= 1e-12
    if N <= 200:
        _, pref = oracle.forces_periodic(x, m, eps, L, G=G, a=a, with_phi=True)
        ep = np.abs(phi.cpu().numpy() - pref)[t] / (G * ps)
        assert ep.max() <= 1e-12
