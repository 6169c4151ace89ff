"""The FFT form of the velocity spectrum at the edges of its ranges: the
switches to and from the direct transform (159 / 160 and 4096 / 4097 rows), the
FFT lengths 512 ... 8192 just below and above their last row count, primes,
tracer counts that do not fill the eight XCDs, and a NaN in one tracer."""
import numpy as np
import pytest

from paper_1208_3444_amd import colatus
from conftest import to_dev

pytestmark = pytest.mark.gpu


def _track(M, T, seed):
    rng = np.random.default_rng(seed)
    n = np.arange(M)[:, None, None]
    v = rng.normal(size=(1, 3, T)) + np.sin(0.3 * n * rng.uniform(size=(1, 3, T)))
    v = v + 0.1 * rng.normal(size=(M, 3, T))
    return np.ascontiguousarray(np.stack([np.cumsum(v, axis=0), v], axis=1))


@pytest.mark.parametrize("remove_mean", [False, True])
@pytest.mark.parametrize("M,T", [(47, 3), (159, 3), (160, 9), (163, 9), (256, 1), (257, 17), (512, 8),
                                 (513, 5), (1001, 7), (1024, 2), (1025, 3), (2048, 2), (2049, 3),
                                 (4096, 2), (4097, 2)])
def test_spectrum_matches_numpy(dev, M, T, remove_mean):
    """Against numpy's FFT.  Rounding of either transform leaves each amplitude
    within a few eps log2(M) of the series' norm, ||w|| = sqrt(M) rms, so each
    power within 2 |F| times that: |dE| <= 2 sqrt(E S) d + S d^2 with S = sum w^2
    the total power of the row, d = 32 eps log2(M) for both transforms."""
    tr = _track(M, T, 7 * M + T)
    got = colatus.velocity_spectrum(to_dev(tr, dev), remove_mean=remove_mean).cpu().numpy()
    w = tr[:, 1]
    if remove_mean:
        w = w - w.mean(axis=0)
    F = np.fft.rfft(w, axis=0)
    ref = (np.abs(F) ** 2).sum(axis=1).T / M
    S = (tr[:, 1] ** 2).sum(axis=(0, 1))[:, None]
    d = 32 * np.finfo(float).eps * np.log2(M)
    bound = 2 * np.sqrt(ref * S) * d + S * d * d
    assert got.shape == ref.shape
    print(f"M={M}: max of |dE| / bound {np.max(np.abs(got - ref) / bound):.3f}", flush=True)
    assert np.all(np.abs(got - ref) <= bound)


def test_nan_stays_with_its_tracer(dev):
    tr = _track(301, 10, 3)
    bad = tr.copy()
    bad[77, 1, 1, 4] = np.nan
    a = colatus.velocity_spectrum(to_dev(tr, dev)).cpu().numpy()
    b = colatus.velocity_spectrum(to_dev(bad, dev)).cpu().numpy()
    assert np.isnan(b[4]).all()
    keep = np.arange(10) != 4
    assert np.array_equal(a[keep], b[keep])
