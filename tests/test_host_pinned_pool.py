"""The pool of pinned host blocks (csrc/pinned_pool.h, plain C++) on the CPU under the
address and undefined-behaviour sanitizers (tests/host/pinned_pool_check.cpp)."""
import os
import shutil
import subprocess

import pytest

from tests.test_host_sanitizers import CSRC, HERE, _run


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_pinned_pool_is_bounded(tmp_path):
    exe = str(tmp_path / "pinned_pool_check")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-omit-frame-pointer",
           "-pthread", "-I" + CSRC, os.path.join(HERE, "host", "pinned_pool_check.cpp"), "-o", exe]
    subprocess.run(cmd, check=True, capture_output=True, text=True)
    _run(exe)
