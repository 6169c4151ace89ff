"""Batches of many tiny boxes: the common masses found by a block per box (2048
boxes at most) and by the passes over all particles, boxes of equal and of
unequal masses mixed."""
import numpy as np
import pytest

from paper_1208_3444_amd import colatus, inputs
from conftest import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-13), ("mixed_twosum", 2e-6)])
@pytest.mark.parametrize("n_boxes", [2048, 2049])
def test_masses_of_many_boxes(dev, n_boxes, prec, tol):
    """Against direct sums, relative to the sum of the pair magnitudes: at most
    eleven terms, each within a few roundings of its type (FP64: 4e-15 of r^-1
    three times over; FP32: 2^-24 in each coordinate and operation, 12 or so)."""
    rng = np.random.default_rng(n_boxes)
    sizes = rng.integers(1, 13, n_boxes)
    off = np.concatenate([[0], np.cumsum(sizes)])
    N, eps = int(off[-1]), np.full(n_boxes, 0.05)
    x = rng.uniform(size=(3, N))
    box = np.repeat(np.arange(n_boxes), sizes)
    m = np.where(box % 3 == 0, rng.uniform(0.5, 1.5, N), 0.5 + box % 5)
    m[off[7]:off[8]] = -1.0  # equal, but not positive
    got = colatus.forces(to_dev(x, dev), to_dev(m, dev), 0.0, precision=prec,
                         batch=(off, eps)).cpu().numpy()
    for b in range(n_boxes):
        s = slice(off[b], off[b + 1])
        d = x[:, None, s] - x[:, s, None]
        w = m[s] * ((d ** 2).sum(0) + 0.05 ** 2) ** -1.5
        mag = (np.abs(w) * np.sqrt((d ** 2).sum(0))).sum(1)
        err = np.linalg.norm(got[:, s] - (w * d).sum(2), axis=0)
        assert (err <= tol * mag + 1e-140).all(), b


@pytest.mark.parametrize("prec", ["fp64", "mixed_twosum"])
@pytest.mark.parametrize("diag", [False, True])
def test_runs_of_many_boxes(dev, prec, diag):
    """The momentum made from the velocity by the integrations themselves (2048
    blocks at most) and by conversions of their own: the same bits."""
    n_boxes, n, few = 2050, 3, 40
    rng = np.random.default_rng(4)
    x, v = rng.uniform(size=(3, n_boxes * n)), 0.1 * rng.normal(size=(3, n_boxes * n))
    m, off = np.full(n_boxes * n, 0.3), np.arange(n_boxes + 1) * n

    def run(k):
        t = [to_dev(np.ascontiguousarray(a[..., :k * n]), dev) for a in (x, v, m)]
        rows = colatus.run(*t, 0.0, 1.0, inputs.LCDM, 0.2, 1.0, 9, first_step=2, last_step=5,
                           precision=prec, batch=(off[:k + 1], np.full(k, 0.05)), diag=diag)
        return t[0].cpu().numpy(), t[1].cpu().numpy(), rows

    colatus.set_option(colatus.OPT_PAIR_FORM, 2)
    try:
        a, b = run(few), run(n_boxes)
    finally:
        colatus.set_option(colatus.OPT_PAIR_FORM, -1)
    assert np.array_equal(a[0], b[0][:, :few * n]) and np.array_equal(a[1], b[1][:, :few * n])
    if diag:
        for r, q in zip(a[2], b[2]):
            assert all(np.array_equal(r[f], q[f]) for f in colatus.DIAG_FIELDS)
