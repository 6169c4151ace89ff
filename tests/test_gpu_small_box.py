"""The one-launch form of small boxes against the general ordered loop
(OPT_PAIR_FORM 0) and the oracle, at sizes around its tiles, rows and limits.

FP32 pairs: the same additions in the same order, so the same bits.  FP64
pairs: sums of N terms in another order, at most N * 2^-53 = 1e-12 of the sum
of magnitudes, compared in the 2-norm at 1e-12."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_1208_3444_amd import colatus, inputs
from conftest import to_dev

pytestmark = pytest.mark.gpu


def _cloud(n, equal):
    x, m = inputs.random_cloud(n, n, scale=0.5)
    return x, (np.full(n, 0.7 / n) if equal else m)


def _both(call):
    small = call()
    colatus.set_option(colatus.OPT_PAIR_FORM, 0)
    try:
        return small, call()
    finally:
        colatus.set_option(colatus.OPT_PAIR_FORM, -1)


def _same(a, b, prec):
    for u, v in zip(a, b):
        if prec == "fp64":
            d = float((u - v).norm())
            assert d <= 1e-12 * float(v.norm()), d
        else:
            assert torch.equal(u, v)


@pytest.mark.parametrize("prec", ["fp64", "mixed_twosum", "mixed_f64acc", "fp32"])
@pytest.mark.parametrize("N", [1, 2, 15, 17, 128, 129, 511, 513, 1000, 2049, 4096, 4097, 6145])
def test_forces_match_the_ordered_loop(dev, N, prec):
    x, m = (to_dev(a, dev) for a in _cloud(N, N % 2 == 0))
    if N == 1:  # exactly zero (the ordered loop's FP64 padding leaves 1e-150)
        assert not any(t.any() for t in colatus.forces(x, m, 0.01, precision=prec, with_phi=True))
        return
    att, bg = (0.3, (0.1, 0.2, -0.1)), (0.2, (0.0, 0.1, 0.0))
    _same(*_both(lambda: (colatus.forces(x, m, 0.01, a=0.5, precision=prec),)), prec)
    _same(*_both(lambda: colatus.forces(x, m, 0.01, a=0.5, precision=prec, with_phi=True)), prec)
    _same(*_both(lambda: colatus.forces(x, m, 0.0, precision=prec, with_phi=True)), prec)
    ext = _both(lambda: colatus.forces(x, m, 0.02, precision=prec, with_phi=True, attractor=att,
                                       background=bg))
    for u, v in zip(*ext):  # the external terms are contracted differently
        assert float((u - v).norm()) <= 1e-12 * float(v.norm())


@pytest.mark.parametrize("prec", ["fp64", "mixed_twosum"])
def test_ragged_boxes_and_oracle(dev, prec):
    sizes = (1, 300, 17, 1290, 128)
    off = np.concatenate([[0], np.cumsum(sizes)])
    eps = np.array([0.01, 0.02, 0.0, 0.03, 0.01])
    x, m = _cloud(int(off[-1]), False)
    m[off[1]:off[2]] = 0.25
    xt, mt = to_dev(x, dev), to_dev(m, dev)
    a, b = _both(lambda: colatus.forces(xt, mt, 0.0, precision=prec, with_phi=True,
                                        batch=(off, eps)))
    _same(a, b, prec)
    if prec == "fp64":
        for k in (1, 3):
            s = slice(off[k], off[k + 1])
            ref = oracle.forces(np.ascontiguousarray(x[:, s]), m[s].copy(), eps[k])
            ref = ref[0] if isinstance(ref, tuple) else ref
            got = a[0].cpu().numpy()[:, s]
            assert np.linalg.norm(got - ref) <= 1e-12 * np.linalg.norm(ref)


@pytest.mark.parametrize("prec", ["fp64", "mixed_twosum"])
def test_runs_and_cached_steps(dev, prec):
    N = 1100
    x, m = (to_dev(a, dev) for a in _cloud(N, True))
    v = 0.1 * torch.randn(3, N, dtype=torch.float64, device=dev,
                          generator=torch.Generator(dev).manual_seed(1))

    def run():
        u, w = x.clone(), v.clone()
        colatus.run(u, w, m, 0.05, 1.0, inputs.LCDM, 0.2, 1.0, 12, precision=prec)
        return u, w

    def steps():
        u, w = x.clone(), v.clone()
        g = colatus.forces(u, m, 0.05, precision=prec)
        for k in range(3):
            colatus.step(u, w, m, 0.05, 1.0, inputs.LCDM, 0.2 + 0.1 * k, 0.3 + 0.1 * k,
                         precision=prec, g_cache=g)
        return u, w, g

    _same(*_both(run), prec)
    _same(*_both(steps), prec)


@pytest.mark.parametrize("prec", ["fp64", "mixed_twosum"])
@pytest.mark.parametrize("first,last", [(0, 1), (0, 2), (3, 8)])
def test_run_in_one_launch_per_step(dev, prec, first, last):
    """Odd and even counts (the positions end in either buffer), tracks, ragged
    boxes; an external term with FP64 pairs (contracted differently)."""
    off, eps = np.array([0, 200, 203, 1100]), np.array([0.05, 0.1, 0.03])
    x, m = (to_dev(a, dev) for a in _cloud(1100, False))
    v = 0.1 * torch.randn(3, 1100, dtype=torch.float64, device=dev,
                          generator=torch.Generator(dev).manual_seed(2))

    def run():
        u, w = x.clone(), v.clone()
        bg = (0.2, (0.0, 0.1, 0.0)) if prec == "fp64" else None
        _, tr = colatus.run(u, w, m, 0.0, 1.0, inputs.LCDM, 0.2, 1.0, 40, first_step=first,
                            last_step=last, precision=prec, batch=(off, eps), background=bg,
                            tracers=[0, 201, 1099])
        return u, w, tr

    _same(*_both(run), prec)


@pytest.mark.parametrize("prec", ["fp64", "mixed_twosum"])
@pytest.mark.parametrize("n", [1, 6])
def test_adjoint_forward_in_one_launch_per_step(dev, prec, n):
    """Every position kept (one launch a step) against checkpoints (two): the
    same bits, with and without the final state."""
    N = 1000
    x, m = (to_dev(a, dev) for a in _cloud(N, False))
    gen = torch.Generator(dev).manual_seed(3)
    v, lx, lv = (torch.randn(3, N, dtype=torch.float64, device=dev, generator=gen)
                 for _ in range(3))
    out = [colatus.adjoint(x, 0.1 * v, m, 0.05, 1.0, inputs.LCDM, 0.2, 1.0, n, lx, lv,
                           checkpoint_every=k, precision=prec, return_state=state)
           for k, state in ((0, True), (n, True), (0, False))]
    for a, b in zip(out[0], out[1]):
        assert torch.equal(a, b)
    for a, b in zip(out[0], out[2]):
        assert torch.equal(a, b)


@pytest.mark.parametrize("prec", ["fp64", "mixed_twosum"])
def test_results_may_replace_the_positions(dev, prec):
    N = 1000
    x, m = (to_dev(a, dev) for a in _cloud(N, True))
    want = colatus.forces(x, m, 0.01, precision=prec)
    buf = x.clone()
    p = ctypes.c_void_p(buf.data_ptr())
    rc = colatus.lib().colatus_forces(p, ctypes.c_void_p(m.data_ptr()), N, 0.01, 1.0, 1.0,
                                      0 if prec == "fp64" else 1, p, None, None, None, None,
                                      ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    assert torch.equal(buf, want)
