"""The streamed lists of the tiled products, checked on the host (no GPU):
`tests/host/stream_check.cpp` builds them with the library's own builder and
walks them as the kernel does."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_streams_walk_to_the_row_sums(tmp_path):
    from paper_1601_08201_amd.build import LIB_PATH, compile_flags, hipcc
    if not os.path.exists(LIB_PATH):
        pytest.skip("library not built")
    exe = str(tmp_path / "stream_check")
    cmd = [hipcc()] + [f for f in compile_flags() if f not in ("-fPIC",)] + [
        "-x", "hip", os.path.join(ROOT, "tests", "host", "stream_check.cpp"),
        "-L" + os.path.dirname(LIB_PATH), "-lsgtv", "-Wl,-rpath," + os.path.dirname(LIB_PATH), "-o", exe]
    subprocess.run(cmd, check=True, capture_output=True, timeout=600)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    print(out.stdout)
    assert out.returncode == 0, out.stdout + out.stderr
    assert out.stdout.strip().endswith("ok")
    assert out.stdout.count("random ") == 24 and out.stdout.count(": streamed") >= 10
