"""The one-sided work lists of the periodic real space (FP32 pairs of small
boxes): coverage on the host, and the field on both sides of the switch to the
pair items against the oracle on the GPU."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIBDIR = os.path.join(ROOT, "paper_1208_3444_amd")


def test_onesided_list_meets_every_ordered_pair_once(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    exe = str(tmp_path / "onesided_check")
    rocm_lib = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "lib")
    cmd = [hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I",
           os.path.join(ROOT, "include"), "-I", os.path.join(LIBDIR, "csrc"),
           os.path.join(ROOT, "tests", "host", "onesided_check.cpp"), "-L", LIBDIR, "-lcolatus",
           "-Wl,-rpath," + LIBDIR, "-L", rocm_lib, "-lrocprofiler-sdk-roctx",
           "-Wl,-rpath," + rocm_lib, "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and "all ok" in r.stdout, r.stdout[-4000:]


# 41 parts of 256 (984 symmetric waves: one-sided items) and 43 (1075: pair
# items), the last part ragged; 65 particles (one full wave and one lane)
@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["mixed_twosum", "fp32"])
@pytest.mark.parametrize("N", [65, 513, 10495, 10753])
def test_periodic_field_on_both_sides_of_the_item_switch(dev, N, prec):
    """Conditioned error (the sum of pair magnitudes as scale) of sampled
    targets: FP32 sums of 256 terms carry at most a few 2^-24 of that scale
    in the mean and the erf approximation 1.5e-7, the bars the repository's
    periodic tests use: median 1e-6, max 1e-4."""
    import oracle
    from paper_1208_3444_amd import colatus, inputs
    from conftest import to_dev
    L, eps = 1.3, 0.004
    x, m = inputs.random_cloud(N, 900 + N, scale=L)
    t = np.sort(np.random.default_rng(N).choice(N, min(N, 128), replace=False))
    ref = oracle.forces_periodic(x, m, eps, L, a=0.8, targets=t)
    acc, phi = colatus.forces_periodic(to_dev(x, dev), to_dev(m, dev), eps, L, a=0.8,
                                       precision=prec, with_phi=True)
    acc0 = colatus.forces_periodic(to_dev(x, dev), to_dev(m, dev), eps, L, a=0.8, precision=prec)
    assert np.array_equal(acc.cpu().numpy(), acc0.cpu().numpy())
    d = x[:, None, :] - x[:, t][:, :, None]
    d -= L * np.rint(d / L)
    r2 = (d ** 2).sum(axis=0)
    r2[np.arange(len(t)), t] = np.inf
    fs = (m[None, :] / (r2 + eps * eps)).sum(axis=1) / 0.8 ** 3
    e = np.linalg.norm(acc.cpu().numpy()[:, t] - ref, axis=0) / fs
    print(f"N={N} {prec}: median {np.median(e):.2e} max {e.max():.2e}", flush=True)
    assert np.median(e) <= 1e-6 and e.max() <= 1e-4
    assert np.isfinite(phi.cpu().numpy()).all()
