"""The coefficients of the FP64 logarithm in csrc/model.h are the ones that
csrc/gen_log1p_coef.py prints."""
import os
import re
import subprocess
import sys

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1304_4334_amd", "csrc")


def test_generator_prints_the_coefficients_of_the_source():
    pytest.importorskip("mpmath")
    src = open(os.path.join(CSRC, "model.h")).read()
    m = re.search(r"kLog1pCoef\[(\d+)\]\s*=\s*\{([^}]*)\}", src)
    have = [float.fromhex(v.strip()) for v in m.group(2).split(",") if v.strip()]
    assert len(have) == int(m.group(1))
    out = subprocess.run([sys.executable, os.path.join(CSRC, "gen_log1p_coef.py")], check=True,
                         capture_output=True, text=True).stdout.splitlines()
    degree, error = re.match(r"// degree (\d+), relative error (\S+) with", out[0]).groups()
    assert [float.fromhex(v.strip().rstrip(",")) for v in out[1:]] == have
    assert int(degree) == len(have) - 1 and float(error) == 1.8e-18
