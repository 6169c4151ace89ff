"""The FP64 adjoint of many cotangents (matrix products over the sources)
against the FP64 oracle: counts around its groups of 16 and its limits, sizes
around its blocks of 64 targets and stages of 16 sources, several boxes,
coincident particles without softening.

Tolerance: each row's error is that of a sum of N products in FP64, at most
N * 2^-53 of the sum of magnitudes, under 1e-12 of the gradient here."""
import numpy as np
import pytest

import oracle
from paper_1208_3444_amd import colatus, inputs
from conftest import to_dev

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


def _cloud(n):
    x, m = inputs.random_cloud(n, n, scale=0.5)
    return x, m * np.random.default_rng(n).uniform(0.5, 2.0, n)


@pytest.mark.parametrize("N,C", [(2, 5), (15, 16), (17, 17), (63, 33), (64, 48), (65, 49),
                                 (1000, 6), (3072, 5), (3073, 13), (3200, 18)])
def test_force_vjp_of_many_cotangents(dev, N, C):
    x, m = _cloud(N)
    eps, G = 0.02, 1.3
    lam = np.random.default_rng(C).standard_normal((C, 3, N))
    got = colatus.force_vjp(to_dev(x, dev), to_dev(m, dev), to_dev(lam, dev), eps, G,
                            precision="fp64").cpu().numpy()
    for c in sorted({0, C // 2, C - 1}):
        assert _rel(got[c], oracle.force_vjp(x, m, lam[c], eps, G=G)) <= 1e-12, c


def test_coincident_particles_without_softening(dev):
    N, C = 130, 18
    x, m = _cloud(N)
    x[:, 70] = x[:, 3]
    lam = np.random.default_rng(0).standard_normal((C, 3, N))
    got, few = (colatus.force_vjp(to_dev(x, dev), to_dev(m, dev), to_dev(lam[:k], dev), 0.0, 1.0,
                                  precision="fp64").cpu().numpy() for k in (C, 4))
    # the oracle divides by zero there: the loop over single cotangents is the reference
    for c in range(4):
        assert _rel(got[c], few[c]) <= 1e-12, c


def test_boxes_of_different_sizes(dev):
    sizes, C, n = (3, 200, 64, 17), 18, 3
    parts = [_cloud(k) for k in sizes]
    x = np.concatenate([p[0] for p in parts], axis=1)
    m = np.concatenate([p[1] for p in parts])
    off = np.concatenate([[0], np.cumsum(sizes)])
    rng = np.random.default_rng(1)
    v = 0.2 * rng.standard_normal(x.shape)
    lx, lv = rng.standard_normal((2, C, 3, x.shape[1]))
    eps = 0.05
    gx, gv = colatus.adjoint(to_dev(x, dev), to_dev(v, dev), to_dev(m, dev), eps, 0.7, inputs.LCDM,
                             0.2, 1.0, n, to_dev(lx, dev), to_dev(lv, dev), precision="fp64",
                             batch=(off, np.full(len(sizes), eps)))
    gx, gv = gx.cpu().numpy(), gv.cpu().numpy()
    for b in range(len(sizes)):
        s = slice(off[b], off[b + 1])
        c = [np.ascontiguousarray(a[..., s]) for a in (x, v, m, lx, lv)]
        rx, rv, _, _ = oracle.adjoint(c[0], c[1], c[2], eps, 0.7, inputs.LCDM, 0.2, 1.0, n, c[3],
                                      c[4])
        assert _rel(gx[..., s], rx) <= 1e-11 and _rel(gv[..., s], rv) <= 1e-11, b
