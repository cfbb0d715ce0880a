"""How many tiles of the adjoint's forward x pass (f_xadj) fit a CU, from the registers the
compiler reports for the kernel the adjoint launches.  The pass waits for its rows, and a
tile holds the same bytes in flight whatever its thread count, so its time goes with the
resident tiles: at one instead of two the pass takes 1.4 times as long.
"""

import re
import subprocess

import pytest

from paper_2603_08892_amd import build

UNIT = """#include "ns_fast_eval.hpp"
namespace nsh {{
auto* adjoint = &adj_eval_fast<typename FastOf<{n}>::type, ns::AOP_HEUN>;
}}
"""
# size: resident tiles
TILES = {144: 4, 160: 2, 192: 2, 216: 2, 256: 2}


@pytest.mark.parametrize("n,tiles", sorted(TILES.items()))
def test_adjoint_tiles_fit(n, tiles, tmp_path):
    src = tmp_path / "unit.hip"
    src.write_text(UNIT.format(n=n))
    cmd = build.compile_command(str(src), str(tmp_path / "unit.o"),
                                ["-I", build.CSRC, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage"])
    out = subprocess.run(cmd, capture_output=True, text=True, check=True).stderr
    found = re.findall(r"Function Name: (\S*f_xadj\S*).*?\bVGPRs: (\d+).*?AGPRs: (\d+)", out, re.S)
    assert len(found) == 1
    name, regs = found[0][0], int(found[0][1]) + int(found[0][2])
    waves = 16 * int(re.search(rf"LinePlanILi{n}ELi(\d+)E", name).group(1)) // 64  # a tile is 16 columns
    simd = min(8, 512 // (-(-regs // 8) * 8))
    assert 4 * simd // waves >= tiles, (name, regs)
