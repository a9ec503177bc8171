"""The HIP sources pass the compiler's checks as the build sets them (one of
them: no pointer is passed on with less alignment than its type promises, as a
16-byte load of rows that start on any element would)."""
import glob
import os
import subprocess

import pytest

from paper_2606_02955_amd import build

SOURCES = sorted(glob.glob(os.path.join(build.PKG, "csrc", "*.hip")))


@pytest.mark.parametrize("src", SOURCES, ids=[os.path.basename(s) for s in SOURCES])
def test_device_side_compiles(src):
    assert "-Werror=align-mismatch" in build.HIPCC_FLAGS
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-O3")]
    res = subprocess.run([build.hipcc(), *flags, "-I", build.INCLUDE, "--cuda-device-only", "-fsyntax-only", src],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
