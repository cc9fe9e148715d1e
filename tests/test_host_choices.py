"""What the library chooses on the host before it launches anything, checked
without a GPU by `tests/host/choice_check.cpp`, which includes the library
source."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_host_choices(tmp_path):
    from paper_1601_08201_amd.build import LIB_PATH, compile_flags, hipcc
    if not os.path.exists(LIB_PATH):
        pytest.skip("library not built")
    exe = str(tmp_path / "choice_check")
    cmd = [hipcc()] + [f for f in compile_flags() if f not in ("-fPIC",)] + [
        "-x", "hip", os.path.join(ROOT, "tests", "host", "choice_check.cpp"),
        "-L" + os.path.dirname(LIB_PATH), "-lsgtv", "-Wl,-rpath," + os.path.dirname(LIB_PATH), "-o", exe]
    subprocess.run(cmd, check=True, capture_output=True, timeout=600)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    print(out.stdout)
    assert out.returncode == 0, out.stdout + out.stderr
    assert out.stdout.strip().endswith("ok")
