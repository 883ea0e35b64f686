"""Tile staging by a workgroup of several waves under ThreadSanitizer, on the
CPU: the staging header compiled against a host model of a workgroup (one
thread per lane), a tile as bytes and then, with a demand past a byte, again
as int16 in the same LDS with the same flag word.  The driver exits non-zero on
a failed expectation, and any pair of accesses that no barrier orders aborts
it."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "sanitize")
CLANG = "/opt/rocm/llvm/bin/clang++"  # the header uses clang's vector and address-space types


def _run(cmd):
    r = subprocess.run(cmd, capture_output=True, text=True, env=dict(os.environ, TSAN_OPTIONS="halt_on_error=1"))
    assert r.returncode == 0, "%s\n%s\n%s" % (" ".join(cmd), r.stdout, r.stderr)
    return r.stdout


def test_staging_of_several_waves(tmp_path):
    if shutil.which(CLANG) is None:
        pytest.skip("%s not available" % CLANG)
    exe = str(tmp_path / "staging_driver")
    _run([CLANG, "-std=c++17", "-fsanitize=thread", "-g", "-O1", "-I", os.path.join(HERE, "host_hip"),
          "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2602_05179_amd", "csrc"),
          os.path.join(HERE, "staging_driver.cpp"), "-pthread", "-o", exe])
    assert "all expectations met" in _run([exe])
