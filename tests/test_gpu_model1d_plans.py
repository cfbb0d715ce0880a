"""Every kernel and plan of the 1D model, all modes and 2/3 of them kept, every scheme: direct
sums with their factors in registers (to 32 points), direct sums over the modes (to 64),
transforms of 128, 256, 512 and 1024 points, convolutions of 256, 512, 1024 and 2048.

Tolerance 1e-12 of the largest coefficient, as in test_gpu_model1d.py: FP64 sums of at most
64 terms or transforms of at most 2048 points against the oracle's transforms, errors of
some 1e-16 times the norm each.
"""

import numpy as np
import pytest

from oracle import nl1d
from test_gpu_model1d import SCHEME_FNS, _close, _dev, _host
from test_gpu_model1d_batches import _schemes, _signals

pytestmark = pytest.mark.gpu

LENGTHS = [32, 34, 64, 66, 126, 128, 254, 256, 258, 510, 512, 514, 1022, 1024]


@pytest.mark.parametrize("n", LENGTHS)
@pytest.mark.parametrize("ct", [2 / 3, 1.0])
def test_plan(n, ct):
    from paper_2603_08892_amd import ns
    print(f"[model1d plan] n={n} ct={ct:.3f}", flush=True)
    model = nl1d.NL1DModel(n, ct)
    s = _signals(n, n, 3) * model.m
    for shift in (0.0, 0.5, 0.137):
        got = _host(ns.model1d_nonlinear(_dev(s), n, ct, shift))
        _close(got, np.stack([model.nl(x, shift) for x in s]), f"shift {shift}")
    for name in SCHEME_FNS:
        sd = _dev(s)
        ns.model1d_step(sd, n, ct, 2e-3, 3, name)
        _close(_host(sd), np.stack([_schemes(model, x, 2e-3, name, 3) for x in s]), name)
