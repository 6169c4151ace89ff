"""FP64 adjoint: a caller's cotangents keep the accuracy of the pair differences
however many are passed, and the matrix form that the exponents' unit
cotangents take agrees with the ordered loop at its edges."""
import numpy as np
import pytest

from paper_1208_3444_amd import colatus, inputs
from conftest import to_dev

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


def _vjp(x, m, lam, eps):
    """sum_j M(d)(m_k lam_j - m_j lam_k) and the sums of its terms' magnitudes, in
    extended precision: rounded to FP64, the two products alone lose what the
    differences keep."""
    x, m, lam = (a.astype(np.longdouble) for a in (x, m, lam))
    d = x[:, None, :] - x[:, :, None]
    s = (d ** 2).sum(0) + eps * eps
    r3, r5 = s ** -1.5, 3.0 * s ** -2.5
    u = m[None, :, None] * lam[:, None, :] - m[None, None, :] * lam[:, :, None]
    du = (d * u).sum(0)
    mag = (r3 * np.sqrt((u ** 2).sum(0)) + r5 * np.abs(du) * np.sqrt((d ** 2).sum(0))).sum(1)
    return (r3 * u - r5 * du * d).sum(2), mag


@pytest.mark.parametrize("C", [1, 4, 6, 13, 18, 48])
def test_smooth_and_uniform_cotangents(dev, C):
    """Equal masses, a clumped cloud.  Bar: N terms added in FP64 (each sum, N u of
    the magnitudes), r^-1 within 4e-15 and so r^-5 within 2e-14 = 180 u, the
    reference's own N u."""
    N, eps = 600, 0.004
    rng = np.random.default_rng(3)
    x = rng.normal(size=(3, N)) * 0.3
    x[:, :200] *= 0.02
    m = np.full(N, 1.0 / N)
    lam = rng.normal(size=(C, 3, N))
    lam[0] = 1.0 + 1e-3 * x
    lam[-1] = 0.75 if C > 1 else lam[0]
    got = colatus.force_vjp(to_dev(x, dev), to_dev(m, dev), to_dev(lam, dev), eps, 1.0,
                            precision="fp64").cpu().numpy()
    if C > 1:
        assert not got[-1].any()  # every difference is exactly zero
    ref, mag = _vjp(x, m, lam[0], eps)
    e = np.abs(got[0] - ref).max(0)
    print(f"C={C}: largest error {(e / mag).max():.2e} of the terms' magnitudes", flush=True)
    assert (e <= (2 * N + 180) * U * mag).all()


def _both(call):
    out = []
    for form in (-1, 0):
        colatus.set_option(colatus.OPT_PAIR_FORM, form)
        try:
            out.append([t.cpu().numpy() for t in call()])
        finally:
            colatus.set_option(colatus.OPT_PAIR_FORM, -1)
    return out


def _same_blocks(call):
    """Blocks that the run has carried far from the identity.  Bar: sums of N terms
    in FP64 over six sweeps, the repository's 1e-11 for adjoints."""
    (_, _, a), (_, _, b) = _both(call)
    assert np.linalg.norm(b - np.eye(3)) > 0.05 * np.linalg.norm(b)
    for t in range(len(b)):
        assert np.linalg.norm(a[t] - b[t]) <= 1e-11 * np.linalg.norm(b[t]), t


@pytest.mark.parametrize("N,T", [(2, 2), (15, 5), (17, 6), (63, 11), (64, 16), (65, 17),
                                 (1000, 2), (3072, 2), (3073, 5), (3200, 16)])
def test_exponents_by_matrix_products(dev, N, T):
    x, m = inputs.random_cloud(N, N, scale=0.5)
    m = m * np.random.default_rng(N).uniform(0.5, 2.0, N)
    tr = np.random.default_rng(T).choice(N, T, replace=T > N)
    args = (to_dev(x, dev), to_dev(np.zeros_like(x), dev), to_dev(m, dev))
    _same_blocks(lambda: colatus.ftle(*args, 0.05, 1.3, inputs.LCDM, 0.1, 1.0, 5, tr,
                                      precision="fp64"))


def test_exponents_by_matrix_products_in_boxes(dev):
    """Ragged boxes; in one, two particles at the same place without softening."""
    sizes = (3, 200, 64, 17, 130)
    off, eps = np.concatenate([[0], np.cumsum(sizes)]), np.array([0.05, 0.04, 0.1, 0.05, 0.0])
    x, m = inputs.random_cloud(int(off[-1]), 8, scale=0.5)
    x[:, off[4] + 70] = x[:, off[4] + 3]
    tr = np.array([0, 2, 3, 202, 203, 266, 267, 283, 300])
    args = (to_dev(x, dev), to_dev(np.zeros_like(x), dev), to_dev(m, dev))
    _same_blocks(lambda: colatus.ftle(*args, 0.0, 0.7, inputs.LCDM, 0.2, 1.0, 1, tr,
                                      precision="fp64", batch=(off, eps)))
