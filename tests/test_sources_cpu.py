"""Rules of the kernel sources that no result shows reliably."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2311_03694_amd", "csrc")


def _code(path):
    with open(path) as f:
        return re.sub(r"//[^\n]*", "", f.read())


@pytest.mark.parametrize("name", ["k_fold.hip", "k_kr.hip", "k_res.hip"])
def test_direct_lds_loads_are_waited_for(name):
    """The barrier that follows direct loads into LDS waits for them first: a barrier alone lets a
    wavefront read words that another one's loads have not written yet."""
    code = _code(os.path.join(CSRC, name))
    loads = [m.end() for m in re.finditer(r"__builtin_amdgcn_global_load_lds\(", code)]
    assert loads
    for at in loads:
        m = re.compile(r"(__syncthreads\w*|__builtin_amdgcn_s_barrier|lds_loads_done)\(").search(code, at)
        assert m and m.group(1) == "lds_loads_done", code[at - 60:at + 40]


def test_every_direct_lds_load_is_in_a_checked_source():
    names = {os.path.basename(p) for p in glob.glob(os.path.join(CSRC, "*")) if "_load_lds(" in _code(p)}
    assert names == {"k_fold.hip", "k_kr.hip", "k_res.hip"}
