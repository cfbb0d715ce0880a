"""The 1D model at lengths of every kind of transform plan: the shortest ones, prime
factors taken as direct sums, and lengths with a larger prime factor (convolution),
against the FP64 oracle.

Tolerance 1e-12 of the largest coefficient, as in test_gpu_model1d.py: FP64 transforms of
at most 2048 points on both sides (an error of a few 1e-16 times the norm each).
"""

import numpy as np
import pytest

from oracle import nl1d
from paper_2603_08892_amd import inputs
from test_gpu_model1d import SCHEME_FNS, _close, _dev, _host

pytestmark = pytest.mark.gpu

LENGTHS = [4, 6, 8, 14, 62, 74, 90, 130, 254, 258, 302, 434, 510, 514, 750, 1006, 1018, 1022]


@pytest.mark.parametrize("n", LENGTHS)
@pytest.mark.parametrize("ct", [2 / 3, 1.0])
def test_lengths(n, ct):
    from paper_2603_08892_amd import ns
    print(f"[model1d length] n={n} ct={ct:.3f}", flush=True)
    model = nl1d.NL1DModel(n, ct)
    kept = np.flatnonzero(model.m)
    s = inputs.model1d_random(n, n, 3, int(kept.max()))
    # entries past the retained modes take no part in an evaluation
    sd = _dev(s)
    for shift in (0.0, 0.5, 0.137):
        got = _host(ns.model1d_nonlinear(sd, n, ct, shift))
        _close(got, np.stack([model.nl(x, shift) for x in s]), f"shift {shift}")
        assert (got[:, 0].imag == 0).all()
    for scheme in ("ps_exact", "ps_approx", "rk4"):
        sd = _dev(s)
        ns.model1d_step(sd, n, ct, 2e-3, 2, scheme)
        want = np.stack([SCHEME_FNS[scheme](model, SCHEME_FNS[scheme](model, x, 2e-3), 2e-3) for x in s])
        _close(_host(sd), want, scheme)


def test_longest_batch_is_independent():
    """A batch of more signals than compute units gives each signal what it gives alone."""
    from paper_2603_08892_amd import ns
    n, b = 74, 600
    s = inputs.model1d_random(n, 5, b, 30)
    all_, one = _dev(s), _dev(s[437:438])
    ns.model1d_step(all_, n, 1.0, 1e-3, 3, "ps_exact")
    ns.model1d_step(one, n, 1.0, 1e-3, 3, "ps_exact")
    assert np.array_equal(_host(all_)[437], _host(one)[0])
