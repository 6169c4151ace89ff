"""The periodic potential (and field beside it) of boxes large enough for the pair
items of the real space, whose reactions carry the sources' part of both: sampled
particles against the oracle.  Sizes just above the switch from the one-sided
items (28 parts of 256 with FP64 pairs, 42 with FP32), the last part ragged."""
import numpy as np
import pytest

import oracle
from paper_1208_3444_amd import colatus, inputs
from conftest import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,prec,order", [(7425, "fp64", "morton"), (7425, "fp64", "random"),
                                          (8193, "fp64", "random"),
                                          (10753, "mixed_twosum", "morton"),
                                          (10753, "mixed_f64acc", "random"),
                                          (10753, "fp32", "random")])
@pytest.mark.parametrize("eps", [0.0, 0.004, 0.2])
def test_potential_of_the_pair_items(dev, N, prec, order, eps):
    """Relative to the sums of the pair magnitudes, the repository's bars: FP64 sums
    of N terms leave a few 1e-16 sqrt(N), within 1e-12; FP32 sums of 256 terms a
    few 2^-24 and the erf approximation 1.5e-7, median 1e-6 and at most 1e-4."""
    L, G, a = 1.6, 1.1, 0.9
    rng = np.random.default_rng(N)
    if order == "random":
        x, m = inputs.random_cloud(N, 70 + N, scale=L)
    else:
        x, m = np.ascontiguousarray(inputs.lcdm_grf(23).x[:, :N]) * L, rng.uniform(0.5, 1.5, N) / N
    t = np.unique(np.concatenate([[0, 63, 64, 255, 256, N - 1, N - N % 256],
                                  rng.choice(N, 60, replace=False)]))
    ref, pref = oracle.forces_periodic(x, m, eps, L, G=G, a=a, targets=t, with_phi=True)
    acc, phi = colatus.forces_periodic(to_dev(x, dev), to_dev(m, dev), eps, L, G=G, a=a,
                                       precision=prec, with_phi=True)
    d = x[:, None, :] - x[:, t][:, :, None]
    d -= L * np.rint(d / L)
    r2 = (d ** 2).sum(axis=0)
    r2[np.arange(len(t)), t] = np.inf
    fs = (m[None, :] / (r2 + eps * eps)).sum(axis=1) * G / a ** 3
    ps = (m[None, :] / np.sqrt(r2 + eps * eps)).sum(axis=1) * G
    e = np.linalg.norm(acc.cpu().numpy()[:, t] - ref, axis=0) / fs
    ep = np.abs(phi.cpu().numpy()[t] - pref) / ps
    print(f"N={N} {prec} {order} eps={eps}: field {e.max():.2e}, potential median "
          f"{np.median(ep):.2e} max {ep.max():.2e}", flush=True)
    if prec == "fp64":
        assert e.max() <= 1e-12 and ep.max() <= 1e-12
    else:
        assert np.median(e) <= 1e-6 and e.max() <= 1e-4
        assert np.median(ep) <= 1e-6 and ep.max() <= 1e-4
