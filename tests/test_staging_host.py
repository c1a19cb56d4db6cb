"""The pinned metadata blocks (paper_2608_11152_amd/csrc/staging.h) built with g++ under the address and
undefined-behaviour sanitizers and driven on stand-ins for streams and events (tests/staging_check.cpp): no piece is
written again before its reader has run, also when streams are destroyed with work pending and their handles given to
new ones; the refusals; the events recorded.  CPU only; no HIP code is built here."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.mark.parametrize("seed", ["1", "2"])
def test_staging_blocks_under_sanitizers(tmp_path, seed):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ is not available")
    exe = str(tmp_path / "staging_check")
    cmd = [cxx, "-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer", "-fsanitize=address,undefined",
           "-fno-sanitize-recover=all", f"-I{os.path.join(ROOT, 'include')}", os.path.join(HERE, "staging_check.cpp"),
           "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe, seed], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "ok: staging blocks" in r.stdout
