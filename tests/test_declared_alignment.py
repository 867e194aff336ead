"""No kernel promises more alignment than its rows have: D and the dense outputs may
start at any element and have any stride, so a pointer to them must not turn into one
to an ordinary 16-byte vector. The compiler says so where it happens."""
import os
import subprocess

import pytest

from paper_1711_05519_amd import build as B


@pytest.mark.parametrize("src", B.SOURCES)
def test_no_pointer_gains_alignment(src):
    cmd = [B.hipcc(), *B.FLAGS, "--cuda-device-only", "-fsyntax-only", "-Werror=align-mismatch",
           os.path.join(B.CSRC, src)]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
