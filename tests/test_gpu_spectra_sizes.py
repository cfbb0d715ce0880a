"""The spectra reduction at sizes where its split of the rows and of k_z changes (one
chunk of 64 k_z and several, full and ragged, the k_z = N/2 column by itself, fewer pairs
of rows than wavefronts), on arbitrary states with every entry non-zero, Nyquist planes
included, against the FP64 oracle.

Tolerance: sums of at most N^3 FP64 terms, 1e-11 of the sum of the terms' absolute values
(energies and dissipation: of the bin itself; transfer and helicity cancel: of the energy
scale).
"""

import numpy as np
import pytest

from oracle import spectra
from test_gpu_parity import _host, _rep, _solver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,prec", [(8, "fp64"), (10, "fp32"), (18, "fp64"), (50, "fp32"), (96, "fp64"),
                                    (128, "fp32"), (150, "fp64"), (160, "fp32"), (256, "fp32"), (270, "fp64")])
@pytest.mark.parametrize("transfer", [False, True])
def test_spectra_any_state(n, prec, transfer):
    from paper_2603_08892_amd import ns
    print(f"[spectra] n={n} {prec} transfer={transfer}", flush=True)
    rng = np.random.default_rng(n)
    shape = (3, n, n, n // 2 + 1)
    u = _rep(rng.standard_normal(shape) + 1j * rng.standard_normal(shape), prec)
    v = _rep(rng.standard_normal(shape) + 1j * rng.standard_normal(shape), prec) if transfer else None
    s = _solver(n, 1.0, prec=prec, nu=0.013)
    ud, vd = s.to_device(u), None if v is None else s.to_device(v)
    got = s.spectra(ud, vd)
    want = spectra.spectra(u, 0.013, v)
    for key in ("e_shell", "d_shell", "e_1d"):
        assert np.abs(got[key] - want[key]).max() <= 1e-11 * np.abs(want[key]).max(), key
        assert (np.abs(got[key] - want[key]) <= 1e-11 * np.abs(want[key])).all(), key
    scale = want["totals"][0] if v is None else np.sqrt(spectra.inner(u, u) * spectra.inner(v, v))
    assert np.abs(got["t_shell"] - want["t_shell"]).max() <= 1e-11 * scale
    gt, wt = got["totals"], want["totals"]
    assert np.allclose(gt[:2], wt[:2], rtol=1e-11, atol=0) and abs(gt[3] - wt[3]) <= 1e-11 * scale
    assert abs(gt[2] - wt[2]) <= 1e-11 * wt[0] * n * np.sqrt(3) / 2
    if n <= 512:
        static = ns.spectra_static(ud, n, 0.013, vd)
        assert all(np.array_equal(static[k], got[k]) for k in got)
    # entries that are not finite are counted and left out: one on each kind of column
    for k, (i, j, kz) in enumerate(((1, 2, 0), (n - 1, 0, n // 2), (n // 2, n // 2, min(3, n // 2 - 1)))):
        ud[k, i, j, kz] = complex(float("nan"), 0.0) if k else complex(0.0, float("inf"))
        u[:, i, j, kz] = 0
    bad = s.spectra(ud, vd, check_finite=False)
    assert bad["totals"][4] == 3
    want = spectra.spectra(u, 0.013)
    assert np.abs(bad["e_1d"] - want["e_1d"]).max() <= 1e-11 * want["e_1d"].max()
