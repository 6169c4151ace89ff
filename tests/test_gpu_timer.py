"""The kernel timer brackets the launches that run without it: the steps of small boxes
stay one launch each, in runs and in the forward pass of the adjoint."""
import pytest
import torch

from paper_1208_3444_amd import colatus, inputs
from conftest import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "mixed_twosum"])
def test_timed_steps_of_small_boxes(dev, prec):
    N, n = 1000, 5
    x, m = (to_dev(a, dev) for a in inputs.random_cloud(N, 9, scale=0.5))
    v = torch.zeros_like(x)
    lam = torch.ones_like(x)[None]

    def calls():
        u, w = x.clone(), v.clone()
        colatus.run(u, w, m, 0.05, 1.0, inputs.LCDM, 0.2, 1.0, n, precision=prec)
        return (u, w) + tuple(colatus.adjoint(x, v, m, 0.05, 1.0, inputs.LCDM, 0.2, 1.0, n, lam,
                                              lam, checkpoint_every=0, precision=prec))

    plain = calls()
    for kind in range(3):
        colatus.timer_read(kind)
    colatus.set_option(colatus.OPT_TIMER, 1)
    try:
        timed = calls()
        counts = [colatus.timer_read(kind) for kind in range(3)]
    finally:
        colatus.set_option(colatus.OPT_TIMER, 0)
    for a, b in zip(plain, timed):
        assert torch.equal(a, b)
    # the run's n steps and closing kick, the adjoint's n forward steps; its n + 1 products
    assert [k for _, k in counts] == [2 * n + 1, n + 1, 0]
    assert counts[0][0] > 0.0
