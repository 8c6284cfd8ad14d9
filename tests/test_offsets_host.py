"""Offsets on the host that decrease by wrapping around 2^32 (no GPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_wrapped_offsets_are_refused(tmp_path):
    exe = str(tmp_path / "offset_wrap")
    src = [os.path.join(ROOT, p) for p in ("paper_2303_06150_amd/csrc/host_checks.cpp", "tests/native/offset_wrap.cpp")]
    subprocess.run(["g++", "-std=c++17", "-O2", "-pthread", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2303_06150_amd", "csrc"), *src, "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
