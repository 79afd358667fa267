"""CPU tests of the device buffers that contexts keep between bootstraps (kept_buffers.h): on
a stand-in device of limited memory, and that every allocation of the library can have
them back.  The C++ test program is built with g++."""
import glob
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "kept_buffers_test.cpp")
CSRC = os.path.join(ROOT, "paper_2607_05920_amd", "csrc")


def test_kept_buffers(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    exe = tmp_path / "kept_buffers_test"
    r = subprocess.run(["g++", "-std=c++17", "-O2", "-pthread", "-I", CSRC, SRC, "-o", str(exe)], capture_output=True,
                       text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "ALL PASSED" in r.stdout, r.stdout + r.stderr


def test_every_allocation_can_have_them_back():
    """One place calls the runtime's allocator; it tries again once they are given back."""
    calls = {}
    for f in glob.glob(os.path.join(CSRC, "*")):
        with open(f) as fh:
            n = len(re.findall(r"\bhipMalloc(?:Async|Managed|FromPoolAsync)?\s*\(", fh.read()))
        if n:
            calls[os.path.basename(f)] = n
    assert calls == {"api.hip": 1}, calls
