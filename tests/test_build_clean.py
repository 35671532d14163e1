"""The HIP sources compile without a warning under the project's own flags."""
import os
import re
import subprocess

import pytest

from paper_2404_14044_amd import build


@pytest.mark.parametrize("source", build.SOURCES)
def test_no_warnings(source):
    res = subprocess.run([build.HIPCC, *build.FLAGS, f"-I{build.INCLUDE}", "-fsyntax-only",
                          os.path.join(build.CSRC, source)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    # (of the sources: the driver's own remarks on its flags carry no place)
    warnings = [line for line in res.stderr.splitlines() if re.search(r":\d+:\d+: warning:", line)]
    assert not warnings, "\n".join(warnings)
