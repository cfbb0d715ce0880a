"""Host-side check of the plans of csrc/ns_size_plans.hpp: every line plan through the
thread-mapping model of test_fft_plans.py, and the launch shapes the kernels assume
(whole wavefronts for the z passes, tiles of at most 1024 threads, whole blocks of
lines, LDS within a block's 160 KB)."""

import os
import re

import numpy as np
import pytest

from test_fft_plans import ROOT, _ept, _run_plan

HEADER = os.path.join(ROOT, "paper_2603_08892_amd", "csrc", "ns_size_plans.hpp")


def _sizes():
    text = open(HEADER).read()
    plan = r"using {} = (LinePlanD?)<(\d+), (\d+), Radices<([\d, ]+)>, Radices<([\d, ]+)>>;\s*"
    pat = re.compile(r"struct SizePlan<(\w+), (\d+)> \{\s*" + "".join(plan.format(p) for p in ("X", "Y", "Z", "ZA"))
                     + r"static constexpr int PZ = (\d+), PZA = (\d+);")
    out = []
    for g in pat.findall(text):
        plans = [(g[2 + 5 * i], int(g[3 + 5 * i]), int(g[4 + 5 * i]), tuple(map(int, g[5 + 5 * i].split(","))),
                  tuple(map(int, g[6 + 5 * i].split(",")))) for i in range(4)]
        out.append((g[0], int(g[1]), plans, int(g[22]), int(g[23])))
    assert len(out) == text.count("struct SizePlan<"), "a plan the pattern does not read"
    listed = re.findall(r"X\((float|double), (\d+)\)", text)
    assert listed == [(t, str(n)) for t, n, _, _, _ in out]
    return out


SIZES = _sizes()


@pytest.mark.parametrize("typ,n,plans,pz,pza", SIZES, ids=[f"{t}-{n}" for t, n, _, _, _ in SIZES])
def test_size_plan(typ, n, plans, pz, pza):
    elem, cols = (8, 16) if typ == "float" else (16, 8)
    rng = np.random.default_rng(n)
    x = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    for kind, m, tpl, inv, fwd in plans:
        assert (kind == "LinePlanD") == (typ == "double") and m == n
        assert np.prod(inv) == n and fwd == tuple(reversed(inv)) and set(inv) <= {2, 3, 4, 5, 6, 8, 9, 10, 12, 16}
    for kind, m, tpl, inv, fwd in set(plans):
        assert _ept(n, tpl, inv) == _ept(n, tpl, fwd)
        assert np.abs(_run_plan(n, tpl, inv, +1, x) - np.fft.ifft(x) * n).max() <= 1e-12 * np.abs(x).sum()
        assert np.abs(_run_plan(n, tpl, fwd, -1, x) - np.fft.fft(x)).max() <= 1e-12 * np.abs(x).sum()
    for i, (kind, m, tpl, inv, fwd) in enumerate(plans[:2]):   # x and y tiles
        assert tpl * cols <= 1024  # one thread block
        assert elem * (n * (cols + 1) + 3 * n + 2 * cols) <= 160 * 1024
    for (kind, m, tpl, inv, fwd), lines in ((plans[2], pz), (plans[3], pza)):
        assert 64 % tpl == 0 and tpl * lines % 64 == 0 and tpl * lines <= 1024 and n * n % lines == 0
        assert elem * (n + lines * (n + n // 16 + 1) + lines * n) <= 160 * 1024
    # the 32-bit byte offsets of the scratch fields and of the caller's components
    pitch = -(-(n // 2 + 1) // cols) * cols
    assert elem * n * n * pitch < 2 ** 32
