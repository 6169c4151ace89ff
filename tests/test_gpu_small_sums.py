"""Sweeps of small boxes that only write sums, FP32 pairs: the ordered loop up to 2048
particles, the form of small boxes beyond, the same bits; a run has the same state
with and without diagnostics."""
import numpy as np
import pytest
import torch

from paper_1208_3444_amd import colatus, inputs
from conftest import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["mixed_twosum", "mixed_f64acc", "fp32"])
@pytest.mark.parametrize("N", [1, 64, 2048, 2049])
def test_sums_by_either_loop(dev, N, prec):
    x, m = (to_dev(a, dev) for a in inputs.random_cloud(N, N, scale=0.5))
    v = 0.1 * torch.randn(3, N, dtype=torch.float64, device=dev,
                          generator=torch.Generator(dev).manual_seed(5))

    def run(**kw):
        u, w = x.clone(), v.clone()
        colatus.run(u, w, m, 0.05, 1.0, inputs.LCDM, 0.2, 1.0, 20, last_step=3, precision=prec, **kw)
        return u, w

    colatus.set_option(colatus.OPT_PAIR_FORM, 0)
    try:
        plain, he = run(), run(scheme="he")
    finally:
        colatus.set_option(colatus.OPT_PAIR_FORM, -1)
    for a, b in ((run(), plain), (run(diag=True), plain), (run(scheme="he"), he)):
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
