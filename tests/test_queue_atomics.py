"""The search's queues take one atomic per wave and batch: the lanes of a wave add to the
same counter, and the compiler makes one addition of theirs, by the first lane, of as many
as there are.  Its assembly is checked, since the source names one addition per lane."""

import re
import shutil

import pytest

from paper_2202_06929_amd import build_lib

pytestmark = pytest.mark.skipif(shutil.which(build_lib.hipcc()) is None, reason="no hipcc")


def test_one_addition_per_wave(tmp_path):
    asm = open(build_lib.device_asm(str(tmp_path))).read()
    kernels = re.findall(r"^(_Z\S*k_search\S*):", asm, re.M)
    assert len(kernels) == 32
    for name in kernels:
        lines = asm[asm.index("\n" + name + ":"):].split(".Lfunc_end")[0].split("\n")
        found = [k for k, line in enumerate(lines) if "global_atomic_add" in line]
        # The extension's blocks (where the lists hold no distances), long and longer lists.
        assert len(found) == (3 if re.search(r"k_searchILi\d+ELb0E", name) else 2), name
        for k in found:
            before = "\n".join(lines[k - 24:k])
            assert "s_bcnt1_i32_b64" in before and "v_mbcnt_hi_u32_b32" in before, (name, lines[k])
