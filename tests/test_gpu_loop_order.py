"""The grouped symmetric sweep picks its pair loop (phased or plain) by its number of
groups and of pairs of parts; both loops give the same bits, so a box's field does
not depend on what else is in the call."""
import numpy as np
import pytest
import torch

from paper_1208_3444_amd import colatus, inputs
from conftest import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "mixed_twosum", "fp32"])
@pytest.mark.parametrize("equal", [True, False])
@pytest.mark.parametrize("n,copies", [(30, 5000), (200, 1100), (700, 700), (5000, 12),
                                      (11500, 2)])
def test_a_box_alone_and_among_others(dev, n, copies, equal, prec):
    """One box by itself (few groups) and in a batch of copies (many): eps 0 and
    not, with the potential and without."""
    x, m = inputs.random_cloud(n, n, scale=0.5)
    m = np.full(n, 0.7 / n) if equal else m
    off = np.arange(copies + 1) * n
    xs, ms = (to_dev(np.tile(a, copies), dev) for a in (x, m))
    x, m = to_dev(x, dev), to_dev(m, dev)
    colatus.set_option(colatus.OPT_PAIR_FORM, 2)
    try:
        for eps in (0.0, 0.02):
            many, phi = colatus.forces(xs, ms, 0.0, precision=prec, with_phi=True,
                                       batch=(off, np.full(copies, eps)))
            only = colatus.forces(xs, ms, 0.0, precision=prec, batch=(off, np.full(copies, eps)))
            one, p1 = colatus.forces(x, m, eps, precision=prec, with_phi=True)
            o1 = colatus.forces(x, m, eps, precision=prec)
            for b in (0, copies - 1):
                s = slice(off[b], off[b + 1])
                assert torch.equal(many[:, s], one) and torch.equal(phi[s], p1)
                assert torch.equal(only[:, s], o1)
    finally:
        colatus.set_option(colatus.OPT_PAIR_FORM, -1)


@pytest.mark.parametrize("prec", ["mixed_twosum", "mixed_f64acc", "fp32"])
@pytest.mark.parametrize("equal", [True, False])
@pytest.mark.parametrize("C,eps", [(1, 0.01), (4, 0.01), (8, 0.01), (8, 0.0)])
def test_adjoint_of_a_box_alone_and_among_others(dev, C, eps, equal, prec):
    """The ordered adjoint loop: 4096 particles (256 blocks) by themselves and 16
    boxes (4096 blocks).  The static step is so short that the positions stay as
    they are, whatever the forward sweep's shape; the cotangents on the velocities
    alone reach the positions' gradients through two transpose products."""
    n, copies, dt = 4096, 16, 1e-18
    x, m = inputs.random_cloud(n, n, scale=0.5)
    m = np.full(n, 0.7 / n) if equal else m
    lam = 1e9 * np.random.default_rng(C).standard_normal((C, 3, n))
    off = np.arange(copies + 1) * n
    static = dict(inputs.LCDM, H0=0.0)

    def grads(k):
        t = [to_dev(np.tile(a, k), dev) for a in (x, 0.0 * x, m, 0.0 * lam, lam)]
        gx, _ = colatus.adjoint(*t[:3], 0.0, 1.0, static, 1.0, dt, 1, *t[3:], precision=prec,
                                batch=(off[:k + 1], np.full(k, eps)))
        return gx

    colatus.set_option(colatus.OPT_PAIR_FORM, 0)
    colatus.set_option(colatus.OPT_TILE_SLICES, 16)
    try:
        one, many = grads(1), grads(copies)
    finally:
        colatus.set_option(colatus.OPT_PAIR_FORM, -1)
        colatus.set_option(colatus.OPT_TILE_SLICES, 0)
    assert float(one.abs().max()) > 1e-10
    assert torch.equal(one, many[..., :n]) and torch.equal(one, many[..., -n:])


FP32_PAIRS = ("mixed_twosum", "mixed_f64acc", "fp32")


@pytest.mark.parametrize("R,tpb,n,copies,prec",
                         [(4, 64, 300, 1200, p) for p in FP32_PAIRS + ("fp64",)] +
                         [(8, 64, 700, 700, p) for p in FP32_PAIRS] +
                         [(4, 128, 700, 700, p) for p in FP32_PAIRS] + [(2, 128, 300, 1200, "fp64")])
def test_single_items_alone_and_among_others(dev, R, tpb, n, copies, prec):
    """The symmetric sweep of one item per workgroup, at its own tile shapes."""
    x, m = inputs.random_cloud(n, n, scale=0.5)
    off = np.arange(copies + 1) * n
    for key, value in ((colatus.OPT_PAIR_FORM, 2), (colatus.OPT_PAIR_GROUP, 0),
                       (colatus.OPT_TILE_R, R), (colatus.OPT_TILE_TPB, tpb)):
        colatus.set_option(key, value)
    try:
        one, p1 = colatus.forces(to_dev(x, dev), to_dev(m, dev), 0.02, precision=prec,
                                 with_phi=True)
        many, phi = colatus.forces(to_dev(np.tile(x, copies), dev), to_dev(np.tile(m, copies), dev),
                                   0.0, precision=prec, with_phi=True,
                                   batch=(off, np.full(copies, 0.02)))
    finally:
        for key, value in ((colatus.OPT_PAIR_FORM, -1), (colatus.OPT_PAIR_GROUP, 1),
                           (colatus.OPT_TILE_R, 0), (colatus.OPT_TILE_TPB, 0)):
            colatus.set_option(key, value)
    assert torch.equal(many[:, :n], one) and torch.equal(phi[-n:], p1)
