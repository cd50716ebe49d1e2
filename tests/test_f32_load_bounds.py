"""Bounds of the fp32 read's buffer loads (CPU: the generated gfx950 code).

A raw buffer load is checked against its resource's size with the lane and
immediate offsets; the scalar offset is not part of that check.  Rows at or
past T rely on it, so no load may carry a scalar offset.  (Their values are
masked, so a load past the end of V changes no result.)  Nor may a load's
resource sit in vector registers: the compiler then loops over its values with
part of the wave, which gave wrong results in the forms that spill.
"""

import os
import re
import subprocess

import pytest

from paper_2602_07160_amd import build


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no hipcc")
def test_loads_are_checked_in_full(tmp_path):
    out = str(tmp_path / "f32.s")
    src = os.path.join(build.CSRC, "fem_softmax_f32.hip")
    subprocess.run([build.HIPCC, *build.CFLAGS, "--offload-device-only", "-S", src, "-o", out],
                   check=True, capture_output=True)
    with open(out) as f:
        code = [x.split(";")[0].strip() for x in f]
    code = [x for x in code if x]
    at = [i for i, x in enumerate(code) if x.startswith("buffer_load_")]
    loads = [code[i] for i in at]
    assert len(loads) > 100
    operand = re.compile(r"s\[\d+:\d+\], (\S+)( offen| offset:\d+)*$")
    assert [x for x in loads if operand.search(x).group(1) != "0"] == []
    assert [code[i] for i in at if "saveexec" in code[i - 1]] == []
