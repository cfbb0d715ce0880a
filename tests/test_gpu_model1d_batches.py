"""The 1D model's choice between direct sums (one or four wavefronts a signal) and
transforms: every side of its lines against the FP64 oracle, the same result alone and in a
large batch, and what a large batch may cost.

Tolerance 1e-12 of the largest coefficient, as in test_gpu_model1d.py: FP64 sums of at most
1024 terms or transforms of at most 2048 points on one side, transforms on the other, errors
of some 1e-16 times the norm.
"""

import numpy as np
import pytest

from oracle import nl1d
from test_gpu_model1d import SCHEME_FNS, _close, _dev, _host

pytestmark = pytest.mark.gpu

# (length, largest kept mode): the shortest and longest lengths of each kind of sum, modes at
# the powers of two the sums' segments change at, points that fill their threads and do not,
# and both sides of the lines to the transforms
CASES = [(34, 1), (34, 16), (36, 2), (48, 15), (50, 16), (62, 30), (64, 31), (64, 2),
         (66, 31), (66, 32), (70, 34), (72, 35), (90, 29), (90, 31), (126, 31), (126, 32), (126, 62), (126, 7), (126, 8),
         (130, 1), (130, 3), (130, 43), (130, 63), (130, 64), (180, 74), (180, 89), (254, 63), (254, 64), (256, 7),
         (258, 6), (258, 63), (258, 64), (258, 96), (258, 128), (384, 95), (510, 127), (510, 128),
         (514, 31), (514, 85), (514, 110), (514, 127), (514, 128), (720, 117), (1022, 60), (1022, 127), (1022, 255)]


def _ct(n, kmax):
    return min(1.0, (kmax + 0.5) * 2 / n)


def _signals(n, seed, batch):
    """Signals 1 + noise, every mode of the same size."""
    rng = np.random.default_rng(seed)
    shape = (batch, n // 2 + 1)
    s = 0.3 * (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)) / np.sqrt(n)
    s[:, 0] = 1.0
    return s


def _schemes(model, x, dt, name, steps):
    for _ in range(steps):
        x = SCHEME_FNS[name](model, x, dt)
    return x


@pytest.mark.parametrize("n,kmax", CASES)
def test_lengths_and_modes(n, kmax):
    from paper_2603_08892_amd import ns
    print(f"[model1d sums] n={n} kmax={kmax}", flush=True)
    ct = _ct(n, kmax)
    model = nl1d.NL1DModel(n, ct)
    assert np.flatnonzero(model.m).max() == kmax
    s = _signals(n, n + kmax, 3)  # entries past the kept modes too
    sd = _dev(s)
    for shift in (0.0, 0.5, 0.137):
        got = _host(ns.model1d_nonlinear(sd, n, ct, shift))
        _close(got, np.stack([model.nl(x, shift) for x in s * model.m]), f"shift {shift}")
        assert (got[:, 0].imag == 0).all() and (got[:, kmax + 1:] == 0).all()
    for name in SCHEME_FNS:
        x = s * model.m
        sd = _dev(x)
        ns.model1d_step(sd, n, ct, 2e-3, 2, name)
        _close(_host(sd), np.stack([_schemes(model, y, 2e-3, name, 2) for y in x]), name)
    # entries past the kept modes pass through a step
    sd = _dev(s)
    ns.model1d_step(sd, n, ct, 2e-3, 1, "rk4")
    assert np.array_equal(_host(sd)[:, kmax + 1:], s[:, kmax + 1:])
    # in place
    sd = _dev(s)
    want = _host(ns.model1d_nonlinear(sd, n, ct, 0.3))
    ns.model1d_nonlinear(sd, n, ct, 0.3, out=sd)
    assert np.array_equal(_host(sd), want)


@pytest.mark.parametrize("n,kmax", [(22, 10), (48, 23), (126, 20), (126, 62), (128, 63), (130, 43), (258, 6), (514, 60)])
def test_alone_as_in_a_batch(n, kmax):
    from paper_2603_08892_amd import ns
    print(f"[model1d batch] n={n} kmax={kmax}", flush=True)
    ct = _ct(n, kmax)
    s = _signals(n, 7, 3000)
    for name in ("rk4", "ps_exact"):
        many, one = _dev(s), _dev(s[1437:1438])
        ns.model1d_step(many, n, ct, 1e-3, 2, name)
        ns.model1d_step(one, n, ct, 1e-3, 2, name)
        assert np.array_equal(_host(many)[1437], _host(one)[0]), name


def _time(n, kmax, batch=40000):
    """Microseconds of one evaluation of a batch, best of five."""
    import torch
    from paper_2603_08892_amd import ns
    s = torch.zeros(batch, n // 2 + 1, dtype=torch.complex128, device="cuda:0")
    out = torch.empty_like(s)
    best = float("inf")
    for _ in range(6):
        start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        for _ in range(10):
            ns.model1d_nonlinear(s, n, _ct(n, kmax), 0.25, out=out)
        stop.record()
        torch.cuda.synchronize()
        best = min(best, 100 * start.elapsed_time(stop))
    return best


def test_large_batches_of_short_signals():
    """48 points against 32, 2.25 times the terms (measured: 1.2 times the time; with all factors
    in registers, two wavefronts a signal: 5 times)."""
    assert _time(48, 23) <= 2.5 * _time(32, 15)


def test_large_batches_with_few_modes():
    """6 modes of 258 points against all 128 (measured: 0.06 of the time; by transforms: the same)."""
    assert _time(258, 6) <= 0.4 * _time(258, 128)
