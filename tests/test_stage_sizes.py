"""The sizes with passes specialised per stage stand in one list, which every dispatch and
unit follows: a context of a size that one of them left out would run the size-generic
passes on its padded planes."""

import glob
import os
import re

from paper_2603_08892_amd import build


def _read(name):
    with open(os.path.join(build.CSRC, name)) as f:
        return f.read()


def test_one_list_of_stage_sizes():
    listed = re.search(r"#define NS_FOR_EACH_STAGE_SIZE\(X\)((?:.*\\\n)*.*\n)", _read("ns_host_impl.hpp")).group(1)
    sizes = [int(n) for n in re.findall(r"X\((\d+)\)", listed)]
    units = [int(re.search(r"fast_(\d+)", f).group(1)) for f in glob.glob(os.path.join(build.CSRC, "fast_*.hip"))]
    assert sizes == sorted(units)
    assert sizes == [int(n) for n in sorted(re.findall(r"using Fast(\d+) = FastCfg<", _read("ns_fast.hpp")), key=int)]
    for n in sizes:
        assert f"({n})" in _read(f"fast_{n}.hip")
    # no dispatch has a list of its own
    for name in ("ns_host.hip", "ns_fast_eval.hpp", "ns_size_eval.hpp"):
        assert not re.search(r"case \d{2,3}:|\bn == \d{2,3}\b|<\d{2,3}, A?OP>|FastOf<\d", _read(name)), name
