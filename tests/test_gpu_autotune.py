"""Autotuning leaves the forms that have one shape alone: small boxes keep their one
launch, the exponents their matrix products, whatever was tuned before."""
import numpy as np
import pytest
import torch

from paper_1208_3444_amd import colatus, inputs
from conftest import to_dev

pytestmark = pytest.mark.gpu


def test_small_boxes_and_exponents(dev):
    # an unusual bucket (37 boxes of 60): what is tuned here stays for the process
    n_boxes, n = 37, 60
    N, off, eps = n_boxes * n, np.arange(n_boxes + 1) * n, np.full(n_boxes, 0.05)
    x, m = (to_dev(a, dev) for a in inputs.random_cloud(N, 6, scale=0.5))
    v = torch.zeros_like(x)
    lam = torch.ones(1, 3, N, dtype=torch.float64, device=dev)

    def calls():
        f = colatus.forces(x, m, 0.0, precision="fp64", batch=(off, eps), with_phi=True)
        g = colatus.adjoint(x, v, m, 0.0, 1.0, inputs.LCDM, 0.3, 1.0, 2, lam, lam,
                            precision="fp64", batch=(off, eps))
        e = colatus.ftle(x, v, m, 0.0, 1.0, inputs.LCDM, 0.3, 1.0, 2, np.arange(16) * 100,
                         precision="fp64", batch=(off, eps))
        return f + tuple(g) + tuple(e)

    plain = calls()
    colatus.set_option(colatus.OPT_AUTOTUNE, 1)
    try:
        first, second = calls(), calls()
    finally:
        colatus.set_option(colatus.OPT_AUTOTUNE, 0)
    for k, (p, a, b) in enumerate(zip(plain, first, second)):
        assert torch.equal(a, b)
        if k in (2, 3):  # the tuned adjoint: other source slices, FP64 sums of 60 terms
            assert float((a - p).norm()) <= 1e-12 * float(p.norm())
        else:
            assert torch.equal(a, p), k
