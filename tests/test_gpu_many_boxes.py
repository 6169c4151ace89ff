"""Batches of many tiny boxes: the common masses found by a block per box (2048
boxes at most) and by the passes over all particles, boxes of equal and of
unequal masses mixed."""
import numpy as np
import pytest

from paper_1208_3444_amd import colatus
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
