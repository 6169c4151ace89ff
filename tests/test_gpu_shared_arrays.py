"""A run whose velocities share memory with the masses: the masses are read until the
last sweep and the velocities written after it, so the state is that of a run on
separate arrays."""
import numpy as np
import pytest
import torch

from paper_1208_3444_amd import colatus, inputs
from conftest import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "mixed_twosum"])
@pytest.mark.parametrize("N,steps,diag", [(1000, 1, False), (1000, 4, False), (3000, 2, True),
                                          (6144, 3, False), (8000, 2, False)])
def test_velocities_over_the_masses(dev, N, steps, diag, prec):
    x, _ = inputs.random_cloud(N, N, scale=0.5)
    shift = N // 2 + 1
    buf = to_dev(np.random.default_rng(N).uniform(0.5, 1.5, 4 * N) / N, dev)
    results = []
    for shared in (True, False):
        b, u = buf.clone(), to_dev(x, dev)
        m, v = b[:N], b[shift:shift + 3 * N].view(3, N)
        if not shared:
            m, v = m.clone(), v.clone()
        colatus.run(u, v, m, 0.05, 1.0, inputs.LCDM, 0.2, 1.0, 20, last_step=steps,
                    precision=prec, diag=diag)
        results.append((u, v.clone()))
    for a, b in zip(*results):
        assert torch.equal(a, b)
